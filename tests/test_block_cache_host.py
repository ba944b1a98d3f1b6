"""The device-block cache against a host model of several devices (host only):
block_cache.hip is compiled here as C++ with a stand-in for the HIP calls it
makes, in which each allocation belongs to the device it was made on."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2010_00409_amd", "csrc")

MODEL = r"""
#pragma once
#include <cstddef>
#include <cstdio>
#include <cstdlib>
#include <map>
typedef int hipError_t;
enum { hipSuccess = 0, hipErrorOutOfMemory = 2, hipErrorInvalidDevice = 101 };
namespace model {
constexpr int NDEV = 2;
constexpr size_t TOTAL = size_t(64) << 30;
struct Alloc { int dev; size_t bytes; };
inline std::map<void*, Alloc> live;             // fake addresses: never read or written
inline size_t used[NDEV];
inline int current = 0, syncs[NDEV], frees = 0;
inline size_t next = 4096;
inline int inside = 0;
struct Inside { Inside() { ++inside; } ~Inside() { --inside; } };
inline void (*on_failure)() = nullptr;          // what another thread does right after a failure
}
inline hipError_t hipGetDevice(int* d) { *d = model::current; return hipSuccess; }
inline hipError_t hipSetDevice(int d) { model::current = d; return hipSuccess; }
inline hipError_t hipGetLastError() { return hipSuccess; }
inline hipError_t hipDeviceSynchronize() { std::puts("breaks other threads' captures"); std::exit(3); }
inline hipError_t hipMemGetInfo(size_t* avail, size_t* total) {
    *total = model::TOTAL;
    *avail = model::TOTAL - model::used[model::current];
    return hipSuccess;
}
inline hipError_t hipMalloc(void** p, size_t b) {
    model::Inside in;
    *p = nullptr;
    if (model::used[model::current] + b > model::TOTAL) {
        if (model::on_failure) model::on_failure();
        return hipErrorOutOfMemory;
    }
    *p = reinterpret_cast<void*>(model::next);
    model::next += b;
    model::live[*p] = {model::current, b};
    model::used[model::current] += b;
    return hipSuccess;
}
inline hipError_t hipFree(void* p) {
    auto it = model::live.find(p);
    if (it == model::live.end()) { std::puts("free of an address that is not live"); std::exit(3); }
    model::used[it->second.dev] -= it->second.bytes;
    ++model::syncs[it->second.dev];
    model::frees += it->second.bytes >= 4096;       // blocks, not what put() frees to wait
    model::live.erase(it);
    return hipSuccess;
}
"""

HEAD = r"""
#include "block_cache.h"
using tf::host::BlockCache;
using tf::host::DeviceBlock;
constexpr size_t MB = size_t(1) << 20, GB = size_t(1) << 30;
#define CHECK(x) do { if (!(x)) { std::printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
int main() {
    BlockCache& c = BlockCache::get();
"""


def run(tmp_path, body, head=""):
    if not shutil.which("g++"):
        pytest.skip("no host compiler")
    inc = tmp_path / "hip"
    inc.mkdir()
    (inc / "hip_runtime.h").write_text(MODEL)
    main = tmp_path / "main.cc"
    main.write_text('#include "block_cache.h"\n' + head + HEAD + body + "    return 0;\n}\n")
    exe = str(tmp_path / "main")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-I", str(tmp_path), "-I", CSRC, "-x", "c++", str(main),
                        os.path.join(CSRC, "block_cache.hip"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_a_block_stays_with_the_device_it_was_allocated_on(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a, b;
    hipSetDevice(1);
    CHECK(c.take(&a, 64 * MB) == hipSuccess && a.dev == 1);
    hipSetDevice(0);
    c.put(a);                                         // destroyed while another device is current
    CHECK(model::syncs[1] == 1 && model::syncs[0] == 0 && model::current == 0);
    CHECK(c.take(&b, 64 * MB) == hipSuccess);
    CHECK(b.dev == 0 && b.ptr != a.ptr && model::live[b.ptr].dev == 0);
    hipSetDevice(1);
    DeviceBlock d;
    CHECK(c.take(&d, 60 * MB) == hipSuccess);         // the kept block, on its own device
    CHECK(d.ptr == a.ptr && d.bytes == 64 * MB && d.dev == 1);
""")


def test_bounds_are_per_device(tmp_path):
    # an eighth of 64 GB is kept on each device; requests on one device do not
    # age the blocks of the other
    run(tmp_path, r"""
    DeviceBlock a[2], b[2];
    for (int d = 0; d < 2; ++d) {
        hipSetDevice(d);
        CHECK(c.take(&a[d], 6 * GB) == hipSuccess);
        CHECK(c.take(&b[d], 5 * GB) == hipSuccess);
    }
    for (int d = 0; d < 2; ++d) c.put(a[d]);
    CHECK(model::frees == 0);
    c.put(b[0]);                                      // 11 GB on device 0: its older block goes
    CHECK(model::frees == 1 && !model::live.count(a[0].ptr) && model::live.count(a[1].ptr));
    hipSetDevice(0);
    for (int i = 0; i < 4; ++i) { DeviceBlock x; CHECK(c.take(&x, 40 * MB) == hipSuccess); }
    CHECK(model::frees == 1);
    DeviceBlock x;
    CHECK(c.take(&x, 40 * MB) == hipSuccess);         // the fifth request that passes it over
    CHECK(model::frees == 2 && !model::live.count(b[0].ptr) && model::live.count(a[1].ptr));
""")


def test_blocks_below_the_bounds_are_freed_at_once(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a, b, big;
    CHECK(c.take(&a, 31 * MB) == hipSuccess);
    c.put(a);
    CHECK(model::frees == 1);
    CHECK(c.take(&b, 9 * GB) == hipSuccess);          // more than an eighth
    c.put(b);
    CHECK(model::frees == 2);
    CHECK(c.take(&a, 64 * MB) == hipSuccess && c.take(&big, 40 * GB) == hipSuccess);
    c.put(a);                                         // less than half of the device is free
    CHECK(model::frees == 3);
    c.put(DeviceBlock{});
""")


def test_an_allocation_that_fails_gets_the_kept_blocks_first(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a, b;
    void* p = nullptr;
    CHECK(c.take(&a, 8 * GB) == hipSuccess);
    c.put(a);
    CHECK(c.alloc(&p, 60 * GB) == hipSuccess && model::frees == 1);
    CHECK(c.alloc(&p, 8 * GB) == hipErrorOutOfMemory);
    CHECK(c.take(&b, 8 * GB) == hipErrorOutOfMemory && !b.ptr);
""")


def test_kept_blocks_go_when_others_fill_the_device_and_on_request(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a, b, x;
    void* others = nullptr;
    CHECK(c.take(&a, 64 * MB) == hipSuccess && c.take(&b, 64 * MB) == hipSuccess);
    c.put(a);
    CHECK(hipMalloc(&others, 40 * GB) == hipSuccess);          // another allocator
    CHECK(c.take(&x, 128 * MB) == hipSuccess);                 // finds none: the kept block goes
    CHECK(model::frees == 1);
    hipFree(others);
    c.put(b);
    CHECK(model::frees == 2 && c.take(&a, 512 * MB) == hipSuccess);
    CHECK(hipMalloc(&others, 40 * GB) == hipSuccess);
    c.put(x);                                                  // and so does b
    CHECK(model::frees == 4 && !model::live.count(b.ptr) && !model::live.count(x.ptr));
    hipFree(others);
    c.put(a);
    CHECK(model::frees == 5 && model::live.count(a.ptr));
    c.clear();
    CHECK(model::frees == 6 && model::live.empty());
""")


def test_nothing_is_kept_or_handed_out_under_a_byte_limit(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a, b;
    CHECK(c.take(&a, 64 * MB) == hipSuccess);
    c.put(a);
    CHECK(model::frees == 0);
    setenv("TFOCUS_MAX_DEVICE_BYTES", "1000000000", 1);
    CHECK(c.take(&b, 60 * MB) == hipSuccess && b.bytes == 60 * MB && b.ptr != a.ptr);
    c.put(b);
    CHECK(model::frees == 1 && !model::live.count(b.ptr));
""")


def test_a_failed_allocation_is_tried_again_after_another_thread_gave_the_blocks_back(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a;
    void* p = nullptr;
    CHECK(c.take(&a, 8 * GB) == hipSuccess);
    c.put(a);
    model::on_failure = [] { model::on_failure = nullptr; BlockCache::get().clear(); };
    CHECK(c.alloc(&p, 60 * GB) == hipSuccess && p);
""")


def test_no_exception_leaves_the_cache_when_host_memory_is_out(tmp_path):
    run(tmp_path, r"""
    DeviceBlock a;
    CHECK(c.take(&a, 64 * MB) == hipSuccess);
    fail_new = true;
    c.put(a);
    fail_new = false;
    CHECK(model::frees == 1 && !model::live.count(a.ptr));
""", head=r"""
#include <cstdlib>
#include <new>
static bool fail_new = false;
void* operator new(std::size_t n) {
    if (fail_new && !model::inside) throw std::bad_alloc();
    return std::malloc(n);
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, std::size_t) noexcept { std::free(p); }
""")
