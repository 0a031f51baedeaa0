// The kept device memory (ftle_memory.h) against a pretend device: the HIP
// calls below stand in for the runtime's.  Prints the first check that fails.
#include "ftle_memory.h"

#include <cstdio>
#include <cstring>
#include <set>

static std::map<void*, size_t> g_held;   // allocations of the pretend device
static size_t g_used = 0, g_capacity = size_t(1) << 40;
static hipError_t g_wait = hipSuccess;   // what a wait returns
static char* g_next = reinterpret_cast<char*>(size_t(1) << 32);

extern "C" {
hipError_t hipGetDevice(int* dev)
{
    *dev = 0;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t bytes)
{
    if (g_used + bytes > g_capacity) return hipErrorOutOfMemory;
    *p = g_next;
    g_next += bytes + 4096;
    g_held[*p] = bytes;
    g_used += bytes;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    auto it = g_held.find(p);
    if (it == g_held.end()) return hipErrorInvalidValue;
    g_used -= it->second;
    g_held.erase(it);
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return g_wait; }
hipError_t hipDeviceSynchronize() { return g_wait; }
}

using namespace ftle;

#define CHECK(x)                                               \
    if (!(x)) {                                                \
        std::printf("%s:%d: %s\n", __FILE__, __LINE__, #x);    \
        return 1;                                              \
    }

static const size_t MiB = size_t(1) << 20;

// An allocation finds the memory that the library keeps, whoever keeps it.
static int out_of_memory()
{
    // 600 MiB idle in the pool of a device of 1000: the scratch needs 700
    g_capacity = 1000 * MiB;
    void* p = nullptr;
    CHECK(pool_alloc(&p, 600 * MiB) == hipSuccess);
    pool_free(p);
    CHECK(kept(0)->pool.idle_bytes >= 600 * MiB);
    ScratchHold h;
    CHECK(scratch_take(700 * MiB, &h) == hipSuccess && h.p && h.cache);
    CHECK(kept(0)->pool.idle_bytes == 0);
    // a second build of 200 MiB beside it, then one of 400 that nothing can serve
    ScratchHold own, none;
    CHECK(scratch_take(200 * MiB, &own) == hipSuccess && own.p && !own.cache);
    CHECK(scratch_take(400 * MiB, &none) == hipErrorOutOfMemory && !none.p);
    scratch_return(own, nullptr);
    scratch_return(h, nullptr);
    // the idle scratch of 700 MiB gives way to a mesh of 600, a busy one does not
    CHECK(pool_alloc(&p, 600 * MiB) == hipSuccess);
    CHECK(kept(0)->scratch.p == nullptr && kept(0)->scratch.bytes == 0);
    CHECK(scratch_take(300 * MiB, &h) == hipSuccess && h.cache);
    void* q = nullptr;
    CHECK(pool_alloc(&q, 200 * MiB) == hipErrorOutOfMemory);
    CHECK(kept(0)->scratch.p == h.p);
    // a scratch that cannot grow is given up whole, and the next build takes it again
    scratch_return(h, nullptr);
    CHECK(scratch_take(500 * MiB, &h) == hipErrorOutOfMemory && !h.p);
    CHECK(!kept(0)->scratch.busy && kept(0)->scratch.bytes == 0);
    CHECK(scratch_take(300 * MiB, &h) == hipSuccess && h.cache);
    scratch_return(h, nullptr);
    pool_free(p);
    release_kept(*kept(0));
    CHECK(g_held.empty() && g_used == 0);
    return 0;
}

// Memory whose kernels could not be waited for is not handed out again.
static int failed_wait()
{
    void *a = nullptr, *b = nullptr;
    CHECK(pool_alloc(&a, 5 * MiB) == hipSuccess);
    g_wait = hipErrorStreamCaptureUnsupported;
    GiveBack()(a);
    CHECK(!g_held.count(a) && kept(0)->pool.idle.empty() && kept(0)->pool.live.empty());
    CHECK(pool_alloc(&b, 5 * MiB) == hipSuccess && b != a);
    // a build's scratch, and the memory of one beside it
    ScratchHold h, own;
    CHECK(scratch_take(MiB, &h) == hipSuccess && scratch_take(MiB, &own) == hipSuccess && !own.cache);
    void *p = h.p, *q = own.p;
    scratch_return(own, nullptr);
    scratch_return(h, nullptr);
    CHECK(!g_held.count(p) && !g_held.count(q) && kept(0)->scratch.bytes == 0 && !kept(0)->scratch.busy);
    CHECK(scratch_take(MiB, &h) == hipSuccess && h.cache && h.p != p && h.p != q);
    // with waits that succeed they are kept
    g_wait = hipSuccess;
    GiveBack()(b);
    p = h.p;
    scratch_return(h, nullptr);
    CHECK(pool_alloc(&a, 5 * MiB) == hipSuccess && a == b);
    CHECK(scratch_take(MiB, &h) == hipSuccess && h.p == p);
    return 0;
}

// The idle memory stays within its bound, the blocks given back first go first,
// and a block serves the next request of its size class.
static int bound()
{
    void* p[40];
    for (int i = 0; i < 40; ++i) CHECK(pool_alloc(&p[i], (60 + i % 3) * MiB) == hipSuccess);
    std::set<void*> all(p, p + 40);
    CHECK(all.size() == 40);
    size_t held = g_used;
    for (int i = 0; i < 40; ++i) {
        const size_t before = kept(0)->pool.idle_bytes;
        pool_free(p[i]);
        CHECK(kept(0)->pool.idle_bytes <= kPoolBound);
        if (before + pool_class(62 * MiB) <= kPoolBound) CHECK(g_used == held);   // nothing freed yet
    }
    size_t idle = 0;
    for (auto& b : kept(0)->pool.idle) idle += b.first;
    CHECK(idle == kept(0)->pool.idle_bytes && idle == g_used && kept(0)->pool.live.empty());
    CHECK(idle + pool_class(62 * MiB) > kPoolBound);
    CHECK(!g_held.count(p[0]) && g_held.count(p[39]));
    const size_t n = kept(0)->pool.idle.size();
    for (size_t i = 0; i < n; ++i) CHECK(kept(0)->pool.idle[i].second == p[40 - n + i]);
    // the last block of the class is taken, another class is not
    void* q = nullptr;
    CHECK(pool_alloc(&q, 60 * MiB) == hipSuccess && q == p[39]);
    pool_free(q);
    CHECK(pool_alloc(&q, 33 * MiB) == hipSuccess && !all.count(q));
    pool_free(q);
    // larger than the bound: not kept
    CHECK(pool_alloc(&q, kPoolBound + MiB) == hipSuccess);
    pool_free(q);
    CHECK(!g_held.count(q) && kept(0)->pool.idle_bytes <= kPoolBound);
    // the classes: at least the request, at most an eighth more
    for (size_t b = 1; b < 4 * MiB; b += 1 + b / 7) CHECK(pool_class(b) >= b && (b < 512 || pool_class(b) <= b + b / 8));
    release_kept(*kept(0));
    CHECK(g_used == 0 && kept(0)->pool.idle_bytes == 0);
    return 0;
}

int main(int argc, char** argv)
{
    const char* name = argc > 1 ? argv[1] : "";
    if (!std::strcmp(name, "out_of_memory")) return out_of_memory();
    if (!std::strcmp(name, "failed_wait")) return failed_wait();
    if (!std::strcmp(name, "bound")) return bound();
    std::printf("no check of that name\n");
    return 2;
}
