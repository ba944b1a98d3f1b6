// Device memory of solvers and batches.
#pragma once
#include <hip/hip_runtime.h>

#include <cstddef>
#include <mutex>
#include <vector>

namespace tf {
namespace host {

// A device allocation with the device that was current when it was made.
struct DeviceBlock {
    void* ptr = nullptr;
    size_t bytes = 0;
    int dev = 0;
};

// Large device allocations of destroyed solvers and batches, kept for the
// next one of about the same size: a freed block's pages are wiped and
// mapped anew at about 35 GB/s, which made the allocation of a 64-window
// batch (19 GB) cost some 15 times its kernels.  A block belongs to the device
// it was allocated on, whichever device is current when its object goes; it
// enters after that device has been synchronised (what hipFree would do), so no
// queued work of any stream still uses it.  Bounds: blocks of 32 MB and more, an
// eighth of a device's memory, and none while less than half of that is free
// (others' allocations come first; looked at whenever a block comes in and
// whenever a request finds none); a block that four later requests on its
// device pass over is given back by the next one, all are when an allocation of
// the library fails, when a surrogate is created (the next consumer of the
// windows a batch made) and by tf_release_memory.  With TFOCUS_MAX_DEVICE_BYTES
// set, objects get exactly the bytes that the limit counts: nothing is kept or
// handed out.  One mutex: any thread may create and destroy objects.
class BlockCache {
public:
    static BlockCache& get();
    // A block of at least `bytes` on the current device.
    hipError_t take(DeviceBlock* block, size_t bytes);
    // Back into the cache (or to the device, where it does not fit the bounds);
    // the caller's current device stays.
    void put(const DeviceBlock& block);
    // Give every kept block back.
    void clear();
    // hipMalloc, with every kept block given back before it reports that the
    // memory is out.
    hipError_t alloc(void** ptr, size_t bytes);

private:
    struct Kept {
        DeviceBlock block;
        int passed;
    };
    std::mutex mu_;
    std::vector<Kept> free_;
    void clear_locked();
    void drop(int dev);          // every kept block of a device
    void put_current(const DeviceBlock& block);
};

}  // namespace host
}  // namespace tf
