#include "block_cache.h"

#include <cstdlib>
#include <new>

namespace tf {
namespace host {

BlockCache& BlockCache::get() {
    static BlockCache* c = new BlockCache();      // lives until the process ends
    return *c;
}

constexpr size_t CACHE_MIN_BLOCK = size_t(32) << 20;

static bool limited() { return std::getenv("TFOCUS_MAX_DEVICE_BYTES") != nullptr; }

void BlockCache::clear_locked() {
    for (const Kept& k : free_) (void)hipFree(k.block.ptr);
    free_.clear();
}

void BlockCache::drop(int dev) {
    for (size_t i = 0; i < free_.size();) {
        if (free_[i].block.dev == dev) {
            (void)hipFree(free_[i].block.ptr);
            free_.erase(free_.begin() + (long)i);
        } else {
            ++i;
        }
    }
}

void BlockCache::clear() {
    std::lock_guard<std::mutex> lk(mu_);
    clear_locked();
}

hipError_t BlockCache::alloc(void** ptr, size_t bytes) {
    hipError_t e = hipMalloc(ptr, bytes);
    if (e != hipErrorOutOfMemory) return e;
    // tried again also where nothing is kept any more: another thread may have
    // given the blocks back since
    std::lock_guard<std::mutex> lk(mu_);
    (void)hipGetLastError();
    clear_locked();
    return hipMalloc(ptr, bytes);
}

hipError_t BlockCache::take(DeviceBlock* block, size_t bytes) {
    *block = DeviceBlock{nullptr, bytes, 0};
    hipError_t e = hipGetDevice(&block->dev);
    if (e != hipSuccess) return e;
    if (bytes < CACHE_MIN_BLOCK || limited()) return alloc(&block->ptr, bytes);
    std::lock_guard<std::mutex> lk(mu_);
    // the smallest block that holds the request with at most a quarter to spare
    size_t best = free_.size();
    for (size_t i = 0; i < free_.size(); ++i) {
        const DeviceBlock& b = free_[i].block;
        if (b.dev == block->dev && b.bytes >= bytes && b.bytes <= bytes + bytes / 4 &&
            (best == free_.size() || b.bytes < free_[best].block.bytes))
            best = i;
    }
    if (best < free_.size()) {
        *block = free_[best].block;
        free_.erase(free_.begin() + (long)best);
        return hipSuccess;
    }
    for (size_t i = 0; i < free_.size();) {
        if (free_[i].block.dev == block->dev && ++free_[i].passed > 4) {
            (void)hipFree(free_[i].block.ptr);
            free_.erase(free_.begin() + (long)i);
        } else {
            ++i;
        }
    }
    size_t avail = 0, total = 0;
    if (!free_.empty() && (hipMemGetInfo(&avail, &total) != hipSuccess || avail < total / 2)) drop(block->dev);
    e = hipMalloc(&block->ptr, bytes);
    if (e == hipErrorOutOfMemory && !free_.empty()) {
        (void)hipGetLastError();
        clear_locked();
        e = hipMalloc(&block->ptr, bytes);
    }
    return e;
}

void BlockCache::put(const DeviceBlock& block) {
    if (!block.ptr) return;
    int dev = block.dev;
    if (hipGetDevice(&dev) != hipSuccess || (dev != block.dev && hipSetDevice(block.dev) != hipSuccess)) {
        (void)hipFree(block.ptr);
        return;
    }
    put_current(block);
    if (dev != block.dev) (void)hipSetDevice(dev);
}

// Waits for all streams of the current device as every hipFree does (its
// implicit synchronisation, whatever is freed: measured with another stream
// busy).  hipDeviceSynchronize would invalidate a graph capture that another
// thread has under way, and every later one there.
static hipError_t wait_for_device() {
    void* p = nullptr;
    const hipError_t e = hipMalloc(&p, 256);
    return e == hipSuccess ? hipFree(p) : e;
}

// put() with the block's device current.
void BlockCache::put_current(const DeviceBlock& block) {
    size_t avail = 0, total = 0;
    if (block.bytes < CACHE_MIN_BLOCK || limited() || wait_for_device() != hipSuccess ||
        hipMemGetInfo(&avail, &total) != hipSuccess || block.bytes > total / 8) {
        (void)hipFree(block.ptr);
        return;
    }
    std::lock_guard<std::mutex> lk(mu_);
    if (avail < total / 2) {
        (void)hipFree(block.ptr);
        drop(block.dev);
        return;
    }
    size_t held = block.bytes;
    for (const Kept& k : free_) held += k.block.dev == block.dev ? k.block.bytes : 0;
    for (size_t i = 0; held > total / 8 && i < free_.size();) {          // the oldest first
        if (free_[i].block.dev == block.dev) {
            held -= free_[i].block.bytes;
            (void)hipFree(free_[i].block.ptr);
            free_.erase(free_.begin() + (long)i);
        } else {
            ++i;
        }
    }
    try {
        free_.push_back({block, 0});
    } catch (const std::bad_alloc&) {        // called from the C entry points
        (void)hipFree(block.ptr);
    }
}

}  // namespace host
}  // namespace tf
