// Device memory that the library keeps between calls: the memory of destroyed
// meshes and of builds (the pool), and the builds' scratch.  Host code; every
// function has internal linkage and concerns the current device.
#pragma once

#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cstddef>
#include <map>
#include <mutex>
#include <utility>
#include <vector>

namespace ftle {
namespace {

// The memory of destroyed meshes (and of a build's own temporaries) is kept
// for the next ones, per device, up to kPoolBound bytes: a program that rebuilds
// its mesh in every frame otherwise pays for mapping and unmapping it each time
// (127 x 113 x 101 points: 0.8 ms to free a mesh, 0.3 to allocate one, of 3.2 ms
// a frame).  A block is kept only when no kernel can still use it
// (release_device waits for the device, a build for its stream; where that wait
// fails the block goes to hipFree) and taken again for a request of the same size
// class (an eighth of a power of two).  Beyond
// the bound the blocks given back first are freed; ftle_release_cached_memory
// frees all of them, and so does an allocation that would fail otherwise.
constexpr int kMaxCachedDevices = 64;
constexpr size_t kPoolBound = size_t(1) << 30;

struct DevPool {
    std::mutex m;
    std::vector<std::pair<size_t, void*>> idle;   // (class size, block), oldest first
    size_t idle_bytes = 0;
    std::map<void*, size_t> live;                 // blocks in use and their class sizes
};

// Scratch device memory of the device mesh builds, kept per device between
// builds and grown when a build needs more, so that a build does not pay for
// allocating and releasing its temporaries each time.  One build at a time
// holds it (a concurrent build on the same device takes memory of its own);
// ftle_release_cached_memory frees it.
struct BuildScratch {
    std::mutex m;
    void* p = nullptr;
    size_t bytes = 0;
    bool busy = false;
};

struct Kept {
    DevPool pool;
    BuildScratch scratch;
};

// Never destroyed: a mesh may outlive static destructors, and the end of the
// process returns the memory anyway.  NULL for a device out of range.
Kept* kept(int dev)
{
    static Kept* const all = new Kept[kMaxCachedDevices];
    return dev >= 0 && dev < kMaxCachedDevices ? all + dev : nullptr;
}

hipError_t current_kept(Kept** k)
{
    int dev = -1;
    const hipError_t e = hipGetDevice(&dev);
    *k = e == hipSuccess ? kept(dev) : nullptr;
    return e;
}

size_t pool_class(size_t bytes)
{
    size_t step = 64;
    while (step * 16 <= bytes) step *= 2;   // 8 to 16 steps: the sizes of one power of two, in eighths
    return (std::max<size_t>(bytes, 1) + step - 1) / step * step;
}

// Frees idle blocks, oldest first, until `keep` bytes are left.
void pool_trim(DevPool& pool, size_t keep)
{
    for (;;) {
        void* p = nullptr;
        {
            std::lock_guard<std::mutex> lk(pool.m);
            if (pool.idle_bytes <= keep || pool.idle.empty()) return;
            p = pool.idle.front().second;
            pool.idle_bytes -= pool.idle.front().first;
            pool.idle.erase(pool.idle.begin());
        }
        (void)hipFree(p);
    }
}

// Frees what is kept and not in use.
void release_kept(Kept& k)
{
    pool_trim(k.pool, 0);
    std::lock_guard<std::mutex> lk(k.scratch.m);
    if (!k.scratch.p || k.scratch.busy) return;
    (void)hipFree(k.scratch.p);
    k.scratch.p = nullptr;
    k.scratch.bytes = 0;
}

// hipMalloc, tried again without the kept memory when there is too little.
// (Takes the locks of Kept: called without any.)
hipError_t device_malloc(Kept* k, void** p, size_t bytes)
{
    hipError_t e = hipMalloc(p, bytes);
    if (e == hipErrorOutOfMemory && k) {
        (void)hipGetLastError();
        release_kept(*k);
        e = hipMalloc(p, bytes);
    }
    return e;
}

hipError_t pool_alloc(void** p, size_t bytes)
{
    *p = nullptr;
    Kept* k = nullptr;
    hipError_t e = current_kept(&k);
    if (e != hipSuccess) return e;
    const size_t size = pool_class(bytes);
    if (!k) return hipMalloc(p, size);
    {
        std::lock_guard<std::mutex> lk(k->pool.m);
        auto& idle = k->pool.idle;
        for (size_t i = idle.size(); i-- > 0;)
            if (idle[i].first == size) {
                k->pool.live[idle[i].second] = size;
                *p = idle[i].second;
                idle.erase(idle.begin() + (std::ptrdiff_t)i);
                k->pool.idle_bytes -= size;
                return hipSuccess;
            }
    }
    e = device_malloc(k, p, size);
    if (e != hipSuccess) return e;
    std::lock_guard<std::mutex> lk(k->pool.m);
    k->pool.live[*p] = size;
    return hipSuccess;
}

// Gives a block back: kept for reuse if `done`, which says that no kernel can
// still use it, else freed.
void pool_free(void* p, bool done = true) noexcept
{
    if (!p) return;
    try {
        Kept* k = nullptr;
        (void)current_kept(&k);
        if (k) {
            {
                std::lock_guard<std::mutex> lk(k->pool.m);
                auto it = k->pool.live.find(p);
                if (it != k->pool.live.end()) {
                    const size_t size = it->second;
                    k->pool.live.erase(it);
                    if (done) {
                        k->pool.idle.push_back({size, p});
                        k->pool.idle_bytes += size;
                        p = nullptr;
                    }
                }
            }
            pool_trim(k->pool, kPoolBound);
        }
    } catch (...) {
    }
    if (p) (void)hipFree(p);
}

// Gives blocks back after waiting for everything on the device.
struct GiveBack {
    const bool done = hipDeviceSynchronize() == hipSuccess;
    void operator()(void* p) const noexcept { pool_free(p, done); }
};

// A build's hold on the scratch, or on memory of its own while another has it.
struct ScratchHold {
    void* p = nullptr;
    BuildScratch* cache = nullptr;
};

hipError_t scratch_take(size_t need, ScratchHold* h)
{
    Kept* k = nullptr;
    const hipError_t e = current_kept(&k);
    if (e != hipSuccess) return e;
    bool mine = false;
    void* small = nullptr;
    if (k) {
        BuildScratch& c = k->scratch;
        std::lock_guard<std::mutex> lk(c.m);
        if (!c.busy) {
            mine = c.busy = true;
            if (c.p && c.bytes >= need) {
                *h = ScratchHold{c.p, &c};
                return hipSuccess;
            }
            small = c.p;
            c.p = nullptr;
            c.bytes = 0;
        }
    }
    if (!mine) return pool_alloc(&h->p, need);
    if (small) (void)hipFree(small);
    void* p = nullptr;
    const hipError_t a = device_malloc(k, &p, need ? need : 16);
    BuildScratch& c = k->scratch;
    std::lock_guard<std::mutex> lk(c.m);
    if (a != hipSuccess) {
        c.busy = false;
        return a;
    }
    c.p = p;
    c.bytes = need;
    *h = ScratchHold{p, &c};
    return hipSuccess;
}

// The build's kernels on s are waited for (also after a failure).
void scratch_return(ScratchHold& h, hipStream_t s) noexcept
{
    const bool done = hipStreamSynchronize(s) == hipSuccess;
    if (!h.cache) {
        pool_free(h.p, done);
    } else {
        std::lock_guard<std::mutex> lk(h.cache->m);
        if (!done) {
            (void)hipFree(h.cache->p);
            h.cache->p = nullptr;
            h.cache->bytes = 0;
        }
        h.cache->busy = false;
    }
    h = ScratchHold{};
}

}  // namespace
}  // namespace ftle
