// The one-ring stencil of a cell mesh built on the GPU: the neighbour
// determination that precedes the FTLE path (Section 2.2 keeps it on the host,
// off the accelerator; the Conclusions list accelerating it as future work).
// Every point's neighbours are the other points sharing a cell with it,
// ascending, each once.  Hand-written kernels, no library sort:
//
//   1. incidence lists in one pass: each cell appends its index to the list
//      of each of its K = dim + 1 points, a list of at most 16 (triangles)
//      or 32 (tetrahedra) entries per point at a fixed place (atomic
//      cursors, one per distinct point of a workgroup, aggregated in LDS
//      first; the order inside a list does not matter; an index outside
//      [0, n) raises the error flag).  When a point has more incident cells
//      than that, or the fixed lists would not be addressable in 32 bits,
//      the lists are packed instead:
//   2. the counts (from the first pass, or from a counting pass) are scanned
//      into each point's incidence offset (scan_tiles / add_partials:
//      2048-element tiles, then the tiles' sums added back), and
//   3. a second pass appends each cell's index to its points' packed lists;
//   4. rows: one lane per point walks its incident cells and collects their
//      points in a sorted list in registers, then stores its count and the list
//      (a fixed kRowCap slots per point in the workspace); the counts are
//      scanned into the row pointers, and a copy moves the lists into place.
//      A point with more than kRowCap - 2 distinct neighbours is handed to a
//      workgroup of its own (long_rows: its candidates sorted by a bitonic
//      network in LDS, duplicates dropped by a flag scan), once to count and
//      once to write.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ftle_device_math.h"
#include "ftle_internal.h"

namespace ftle {
namespace {

constexpr int kScanThreads = 256, kScanItems = 8, kScanTile = kScanThreads * kScanItems;
constexpr int kRowThreads = 128;   // lanes per workgroup of the row passes
constexpr int kRowCap = 32;        // list entries a lane keeps in registers (the point and one free among them)
constexpr int kLongCap = 4096;     // candidates (with repeats) of a long row
constexpr uint32_t kIncCap2 = 16, kIncCap3 = 32;   // fixed incidence list length (triangles, tetrahedra)

inline unsigned blocks_for(int64_t m, int per = 256) { return (unsigned)((m + per - 1) / per); }

// The points of cell c (tetrahedra: one 16-byte load when the array is
// 16-byte aligned, a workgroup-uniform test).
template <int K>
__device__ inline void load_cell(const int32_t* __restrict__ cells, int64_t c, int32_t (&v)[K])
{
    if (K == 4 && (reinterpret_cast<uintptr_t>(cells) & 15) == 0) {
        const int4 q = reinterpret_cast<const int4*>(cells)[c];
        v[0] = q.x, v[1] = q.y, v[2] = q.z;
        if constexpr (K == 4) v[3] = q.w;
    } else {
#pragma unroll
        for (int a = 0; a < K; ++a) v[a] = cells[c * K + a];
    }
}

// 1 and 3.  A workgroup takes kAggCells cells per lane and first gathers their
// points' occurrences in an LDS hash table (open addressing, keys inserted by
// compare-and-swap), so that each distinct point of the workgroup's cells
// costs one global atomic instead of one per occurrence: cells come in mesh
// order, and neighbouring cells share most of their points.  A point that
// finds no slot within kProbes probes goes to global memory directly.
// The pass waits for those atomics' round trips (83 % of its wave cycles), so
// the used slots are listed as they fill and a lane has one or two atomics one
// after the other instead of one per slot of the table: 127 x 113 x 101 points
// 310 -> 185 us, 1023 x 769 triangle mesh 78 -> 33.  512 threads of two cells
// and 8192 slots: 1024 threads of one cell take 152 us there but lose on cells
// in random order (every point distinct; 70^3: 620 us as before, 707 with
// 1024, 560 with 512).
//   kCount:  cnt[v] += occurrences of v (a cell with an index outside [0, n)
//            sets bit 1 of *err and adds nothing);
//   kPacked: each occurrence of v gets a position from cur[v] (the workgroup
//            reserves its block of positions with one atomic) and
//            inc[position] = its cell;
//   kFixed:  as kCount, and each occurrence of v also gets list position
//            k = the count before it, inc[v cap + k] = its cell while k < cap
//            (beyond it, bit 4 of *err and no store).
constexpr int kAggThreads = 512, kAggCells = 2, kAggSlots = 8192, kProbes = 16;
enum IncMode { kCount, kPacked, kFixed };

__device__ inline uint32_t agg_hash(int32_t v) { return ((uint32_t)v * 2654435761u) >> 19; }   // 13 bits

template <int K, int MODE>
__global__ void __launch_bounds__(kAggThreads) incidence_pass(const int32_t* __restrict__ cells, int64_t n_cells,
                                                              int64_t n, uint32_t* __restrict__ cnt,
                                                              int32_t* __restrict__ inc, int* __restrict__ err,
                                                              uint32_t cap)
{
    constexpr bool FILL = MODE != kCount;
    static_assert(kAggSlots == 1 << 13, "agg_hash gives 13 bits");
    __shared__ int32_t key[kAggSlots];
    __shared__ uint32_t num[kAggSlots];
    __shared__ uint16_t used[kAggThreads * kAggCells * K];   // the slots in use
    __shared__ int n_used;
    const int t = (int)threadIdx.x;
    for (int i = t; i < kAggSlots; i += kAggThreads) {
        key[i] = -1;
        num[i] = 0;
    }
    if (t == 0) n_used = 0;
    __syncthreads();
    // each XCD takes a contiguous stretch of cells (its L2 then holds their points' counters)
    const int64_t c0 = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * (kAggThreads * kAggCells);
    int slot[kAggCells][K];
    uint32_t local[kAggCells][K];
#pragma unroll
    for (int q = 0; q < kAggCells; ++q) {
        const int64_t c = c0 + q * kAggThreads + t;
        int32_t v[K];
        bool ok = c < n_cells;
        if (ok) {
            load_cell<K>(cells, c, v);
#pragma unroll
            for (int a = 0; a < K; ++a) ok &= (uint64_t)(int64_t)v[a] < (uint64_t)n;
            if (MODE != kPacked && !ok) atomicOr(err, 1);
        }
#pragma unroll
        for (int a = 0; a < K; ++a) {
            slot[q][a] = -2;   // nothing to do
            if (!ok) continue;
            uint32_t h = agg_hash(v[a]);
            int s = -1;
            for (int p = 0; p < kProbes; ++p, h = (h + 1) & (kAggSlots - 1)) {
                const int32_t k = atomicCAS(&key[h], -1, v[a]);
                if (k == -1) used[atomicAdd(&n_used, 1)] = (uint16_t)h;
                if (k == -1 || k == v[a]) {
                    s = (int)h;
                    break;
                }
            }
            slot[q][a] = s;
            if (s >= 0) {
                local[q][a] = atomicAdd(&num[s], 1u);
            } else if (MODE == kPacked) {
                inc[atomicAdd(&cnt[v[a]], 1u)] = (int32_t)c;
            } else if (MODE == kFixed) {
                const uint32_t k = atomicAdd(&cnt[v[a]], 1u);
                if (k < cap)
                    inc[(uint32_t)v[a] * cap + k] = (int32_t)c;
                else
                    atomicOr(err, 4);
            } else {
                atomicAdd(&cnt[v[a]], 1u);
            }
        }
    }
    __syncthreads();
    // (over the used slots, not the table: a global atomic's round trip is
    // several microseconds here, and a lane has three of them, not sixteen)
    for (int j = t; j < n_used; j += kAggThreads) {
        const int i = used[j];
        if (FILL)
            num[i] = atomicAdd(&cnt[key[i]], num[i]);   // the block's first position
        else
            atomicAdd(&cnt[key[i]], num[i]);
    }
    if constexpr (MODE == kPacked) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < kAggCells; ++q)
#pragma unroll
            for (int a = 0; a < K; ++a)
                if (slot[q][a] >= 0) inc[num[slot[q][a]] + local[q][a]] = (int32_t)(c0 + q * kAggThreads + t);
    } else if constexpr (MODE == kFixed) {
        __syncthreads();
        bool over = false;
#pragma unroll
        for (int q = 0; q < kAggCells; ++q)
#pragma unroll
            for (int a = 0; a < K; ++a)
                if (slot[q][a] >= 0) {
                    const uint32_t k = num[slot[q][a]] + local[q][a];
                    if (k < cap)
                        inc[(uint32_t)key[slot[q][a]] * cap + k] = (int32_t)(c0 + q * kAggThreads + t);
                    else
                        over = true;
                }
        if (over) atomicOr(err, 4);
    }
}

// ---------------------------------------------------------------------------
// Exclusive scan of m uint32 counts into out[0..m) (Out: uint32 or int64),
// with out[m] = the total.  scan_tiles scans each 2048-element tile and
// writes its sum to partial[tile]; add_partials adds each tile's offset, the
// sum of the tiles before it, which each of its workgroups adds up itself
// (DIRECT) or takes from the partial sums scanned in between by one workgroup
// (scan_partials: chunks of 1024 with a carry).
//
// Bound by launches where it is short, by its bytes where it is long: the
// counts and the results pass through LDS, so that loads and stores are of
// consecutive elements, and sums move by lane shuffles.  787k counts to int64
// 17.3 -> 11.6 us and a launch less, 1.45 M 24.4 -> 16.9 us, 4.1 M 49 -> 23 us.
// ---------------------------------------------------------------------------
template <typename Out>
__device__ inline Out block_inclusive_scan(Out v, Out* s, int tid, int nthreads)
{
    s[tid] = v;
    __syncthreads();
    for (int off = 1; off < nthreads; off <<= 1) {
        const Out t = tid >= off ? s[tid - off] : Out(0);
        __syncthreads();
        s[tid] += t;
        __syncthreads();
    }
    return s[tid];
}

template <typename Out>
__device__ inline Out lane_up(Out v, int by)
{
    if constexpr (sizeof(Out) == 8)
        return (Out)__shfl_up((long long)v, by);
    else
        return (Out)__shfl_up((unsigned int)v, by);
}

template <typename Out>
__global__ void __launch_bounds__(kScanThreads) scan_tiles(const uint32_t* in, int64_t m, Out* out,
                                                             Out* __restrict__ partial, Out* copy)   // in and out may coincide
{
    constexpr int kPad = kScanItems + 1;   // a lane's items, one word apart from the next lane's
    __shared__ Out s[kScanThreads * kPad];
    __shared__ Out wave_sum[kScanThreads / 64];
    const int tid = (int)threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t base = (int64_t)blockIdx.x * kScanTile;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int e = k * kScanThreads + tid;
        s[e / kScanItems * kPad + e % kScanItems] = base + e < m ? (Out)in[base + e] : Out(0);
    }
    __syncthreads();
    Out v[kScanItems], sum = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        v[k] = s[tid * kPad + k];
        sum += v[k];
    }
    Out incl = sum;
    for (int by = 1; by < 64; by <<= 1) {
        const Out u = lane_up(incl, by);
        if (lane >= by) incl += u;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    for (int w = 0; w < wave; ++w) incl += wave_sum[w];
    Out run = incl - sum;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        s[tid * kPad + k] = run;
        run += v[k];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int e = k * kScanThreads + tid;
        if (base + e < m) out[base + e] = s[e / kScanItems * kPad + e % kScanItems];
    }
    if (tid == kScanThreads - 1) {
        partial[blockIdx.x] = incl;
        if (gridDim.x == 1) {
            out[m] = incl;
            if (copy) *copy = incl;
        }
    }
}

template <typename Out>
__global__ void __launch_bounds__(1024) scan_partials(Out* __restrict__ partial, int64_t np, Out* __restrict__ total,
                                                      Out* copy)
{
    __shared__ Out s[1024];
    const int tid = (int)threadIdx.x;
    Out carry = 0;
    for (int64_t c0 = 0; c0 < np; c0 += 1024) {
        const int64_t i = c0 + tid;
        const Out v = i < np ? partial[i] : Out(0);
        const Out incl = block_inclusive_scan<Out>(v, s, tid, 1024);
        if (i < np) partial[i] = carry + incl - v;
        carry += s[1023];
        __syncthreads();
    }
    if (tid == 0) {
        *total = carry;
        if (copy) *copy = carry;
    }
}

// A workgroup per tile.
template <typename Out, bool DIRECT>
__global__ void __launch_bounds__(kScanThreads) add_partials(Out* __restrict__ out, int64_t m,
                                                             const Out* __restrict__ partial, Out* copy)
{
    __shared__ Out wave_sum[kScanThreads / 64];
    const int tid = (int)threadIdx.x;
    const int64_t tile = blockIdx.x;
    Out add = 0;
    if constexpr (DIRECT) {
        for (int64_t p = tid; p < tile; p += kScanThreads) add += partial[p];
        for (int by = 1; by < 64; by <<= 1) {
            const Out u = lane_up(add, by);
            if ((tid & 63) >= by) add += u;
        }
        if ((tid & 63) == 63) wave_sum[tid >> 6] = add;
        __syncthreads();
        add = 0;
#pragma unroll
        for (int w = 0; w < kScanThreads / 64; ++w) add += wave_sum[w];
        if (tid == 0 && tile == (int64_t)gridDim.x - 1) {
            out[m] = add + partial[tile];
            if (copy) *copy = add + partial[tile];
        }
    } else {
        add = partial[tile];
    }
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        const int64_t i = tile * kScanTile + k * kScanThreads + tid;
        if (i < m) out[i] += add;
    }
}

// Tiles up to which each workgroup adds up the sums before it: its reads grow
// with the square of the tiles, the scan in between costs a launch and a serial
// chain (int64, direct / scanned: 44 tiles 7.0 / 9.6 us, 1024 13.7 / 15.7, 4096
// 41.4 / 47.7, 8192 82.6 / 88.8, 16384 268 / 208; uint32 at 8192 63.0 / 60.4).
constexpr int64_t kDirectTiles = 4096;

// copy: another place for the total, or null.
template <typename Out>
hipError_t exclusive_scan(const uint32_t* in, int64_t m, Out* out, Out* partial, hipStream_t stream,
                          Out* copy = nullptr)
{
    const int64_t tiles = (m + kScanTile - 1) / kScanTile;
    const dim3 grid((unsigned)tiles), block(kScanThreads);
    if (tiles > 0) hipLaunchKernelGGL((scan_tiles<Out>), grid, block, 0, stream, in, m, out, partial, copy);
    if (tiles > kDirectTiles || tiles == 0)
        hipLaunchKernelGGL((scan_partials<Out>), dim3(1), dim3(1024), 0, stream, partial, tiles, out + m, copy);
    if (tiles > kDirectTiles)
        hipLaunchKernelGGL((add_partials<Out, false>), grid, block, 0, stream, out, m, (const Out*)partial, copy);
    else if (tiles > 1)
        hipLaunchKernelGGL((add_partials<Out, true>), grid, block, 0, stream, out, m, (const Out*)partial, copy);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// 4. rows.  Lane r (point r) collects its distinct neighbours, at most kRowCap - 2,
// sets deg[r] to their count and stores them, ascending, at store[k * n + r]
// (entry-major, so that each store instruction writes consecutive points).  A
// point with more is appended to longs (deg[r] = 0 until long_rows counts it).
// ---------------------------------------------------------------------------
// Point r's incidence list: inc[p0, p1).  *capp = 0: packed lists at the
// offsets off[r], off[r + 1]; otherwise fixed lists of *capp entries, off[r]
// of them used.
struct IncRange {
    uint32_t p0, p1;
};
__device__ inline IncRange inc_range(const uint32_t* __restrict__ off, uint32_t cap, int64_t r)
{
    if (cap) {
        const uint32_t p0 = (uint32_t)r * cap;
        return IncRange{p0, p0 + off[r]};
    }
    return IncRange{off[r], off[r + 1]};
}

// The list lives in registers, the point itself among its entries (so that it
// counts as found): every candidate is compared with all N entries and, where
// some lane's is new, inserted by one v_med3 per entry, without a branch or a
// memory access per lane.  127 x 113 x 101 points: 304 -> 155 us; 1023 x 769
// triangle mesh 44 -> 27.  (A sorted list in LDS, searched by bisection and
// moved up entry by entry, waited on LDS for 61 % of its cycles and executed
// 4400 vector instructions a wave at 24 cells a point; now 2900.)
//
// N = 16 serves waves whose points have at most 14 neighbours by the count of
// their incident cells (a closed fan of m triangles has m other points, a
// closed ball of m tetrahedra m / 2 + 2); a list that fills up (a point on the
// boundary has more) is collected again with N = 32.
constexpr uint32_t kNone = 0xffffffffu;

// The points of kBatch cells into the list.
template <int K, int N, int BATCH>
__device__ inline void collect_cells(const int32_t* __restrict__ cells, const int32_t (&c)[BATCH], uint32_t (&s)[N])
{
    int32_t v[BATCH][K];
#pragma unroll
    for (int q = 0; q < BATCH; ++q) load_cell<K>(cells, c[q], v[q]);
#pragma unroll
    for (int q = 0; q < BATCH; ++q)
#pragma unroll
        for (int a = 0; a < K; ++a) {
            uint32_t u = (uint32_t)v[q][a];
            bool f[4] = {false, false, false, false};   // four short chains
#pragma unroll
            for (int k = 0; k < N; ++k) f[k & 3] |= s[k] == u;
            const bool found = (f[0] | f[1]) | (f[2] | f[3]);
            if (__ballot(!found) == 0) continue;   // nothing new in the wave
            u = found ? kNone : u;
            // s'[k] = the median of s[k - 1] <= s[k] and u (kNone changes nothing;
            // a full list drops its last entry)
#pragma unroll
            for (int k = N - 1; k > 0; --k) asm("v_med3_u32 %0, %1, %2, %0" : "+v"(s[k]) : "v"(s[k - 1]), "v"(u));
            s[0] = min(s[0], u);
        }
}

// The list of point r from its incidence list, eight cells at a time: their
// loads are issued together (a cell past the end repeats the last one, whose
// points are then found).
template <int K, int N>
__device__ inline void collect_row(const int32_t* __restrict__ cells, const int32_t* __restrict__ inc, uint32_t cap,
                                   uint32_t p0, uint32_t p1, uint32_t r, uint32_t (&s)[N])
{
    constexpr int kBatch = 8;
    constexpr uint32_t kCap = K == 4 ? kIncCap3 : kIncCap2;
    s[0] = r;
#pragma unroll
    for (int k = 1; k < N; ++k) s[k] = kNone;
    if (p1 <= p0) return;
    if (cap == kCap) {
        // a fixed list, 64 or 128 bytes a lane: read whole, before the cells are.
        // (Read in eights between the gathers, the lists' lines left L2, where
        // up to 24 points share a cell, before they were used up: 1.0 GB fetched
        // instead of 0.46.)
        typedef int32_t int4v __attribute__((ext_vector_type(4), aligned(4)));   // a caller's workspace may be unaligned
        int32_t c[kCap];
        const int4v* src = reinterpret_cast<const int4v*>(inc + p0);
#pragma unroll
        for (uint32_t q = 0; q < kCap / 4; ++q) {
            const int4v w = src[q];
#pragma unroll
            for (int e = 0; e < 4; ++e) c[4 * q + e] = w[e];
        }
        const uint32_t m = p1 - p0;
#pragma unroll
        for (uint32_t g = 0; g < kCap; g += kBatch)
            if (__ballot(g < m) != 0) {
                int32_t b[kBatch];
#pragma unroll
                for (int q = 0; q < kBatch; ++q) b[q] = g + q < m ? c[g + q] : c[0];
                collect_cells<K, N>(cells, b, s);
            }
        return;
    }
    for (uint32_t p = p0; p < p1; p += kBatch) {
        int32_t b[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) b[q] = inc[min(p + q, p1 - 1)];
        collect_cells<K, N>(cells, b, s);
    }
}

// The list (less the point itself) to its place; false when it filled up.
template <int N>
__device__ inline bool keep_row(const uint32_t (&s)[N], int64_t n, int64_t r, uint32_t* __restrict__ deg,
                                int32_t* __restrict__ store)
{
    if (s[N - 1] != kNone) return false;
    uint32_t cnt = 0;
#pragma unroll
    for (int k = 1; k < N; ++k) cnt += s[k] != kNone ? 1u : 0u;
    deg[r] = cnt;
#pragma unroll
    for (int k = 0; k < N - 1; ++k)
        if ((uint32_t)k < cnt) store[k * n + r] = (int32_t)(s[k] < (uint32_t)r ? s[k] : s[k + 1]);
    return true;
}

// (Occupancy: 124 and 84 registers; with the scheduler's own choice it hoists
// loads until two waves fit a SIMD, with more waves L2 holds fewer of the cells.)
template <int K>
__global__ void __launch_bounds__(kRowThreads) __attribute__((amdgpu_waves_per_eu(K == 4 ? 4 : 5)))
ring_rows(const int32_t* __restrict__ cells, const int32_t* __restrict__ inc, const uint32_t* __restrict__ off,
          const uint32_t* __restrict__ capp, int64_t n, uint32_t* __restrict__ deg, int32_t* __restrict__ store,
          uint32_t* __restrict__ longs, uint32_t* __restrict__ n_long)
{
    static_assert(kRowCap == 32, "the stored lists hold what a list of 32 registers does");
    // XCD-contiguous rows
    const int64_t r = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * kRowThreads + threadIdx.x;
    if (r >= n) return;
    const uint32_t cap = *capp;
    const IncRange ir = inc_range(off, cap, r);
    bool done = false;
    if (__ballot(ir.p1 - ir.p0 > (K == 4 ? 24u : 14u)) == 0) {
        uint32_t s[16];
        collect_row<K, 16>(cells, inc, cap, ir.p0, ir.p1, (uint32_t)r, s);
        done = keep_row<16>(s, n, r, deg, store);
    }
    if (!done) {
        uint32_t s[kRowCap];
        collect_row<K, kRowCap>(cells, inc, cap, ir.p0, ir.p1, (uint32_t)r, s);
        if (!keep_row<kRowCap>(s, n, r, deg, store)) {
            longs[atomicAdd(n_long, 1u)] = (uint32_t)r;
            deg[r] = 0;
        }
    }
}

// The stored lists into place: col[row_ptr[r] + k] = store[k * n + r] for the
// rows ring_rows kept (a long row's count, set by long_rows, exceeds kRowCap - 2).
// A workgroup's 256 rows are one contiguous stretch of col: each lane puts its
// row into that stretch in LDS (long rows' entries marked -1), then the
// stretch goes out with consecutive lanes writing consecutive entries.  A
// stretch longer than kCopySeg entries (long rows in the workgroup) is
// written row by row instead.
constexpr int kCopySeg = 256 * 24;

__global__ void __launch_bounds__(256) copy_rows(const int32_t* __restrict__ store, int64_t n,
                                                 const uint32_t* __restrict__ deg,
                                                 const int64_t* __restrict__ row_ptr, int32_t* __restrict__ col)
{
    __shared__ int32_t seg[kCopySeg];
    const int t = (int)threadIdx.x;
    const int64_t r0 = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * 256, r = r0 + t;
    const int64_t r1 = min(r0 + 256, n);
    const int64_t base = row_ptr[r0], total = row_ptr[r1] - base;
    const bool live = r < n;
    const uint32_t d = live ? deg[r] : 0u;
    const bool kept = d <= (uint32_t)kRowCap - 2;
    if (total > kCopySeg) {   // workgroup-uniform
        if (live && kept) {
            int32_t* out = col + row_ptr[r];
            for (uint32_t k = 0; k < d; ++k) out[k] = store[(int64_t)k * n + r];
        }
        return;
    }
    if (live) {
        int32_t* dst = seg + (row_ptr[r] - base);
        if (kept)
            for (uint32_t k = 0; k < d; ++k) dst[k] = store[(int64_t)k * n + r];
        else
            for (uint32_t k = 0; k < d; ++k) dst[k] = -1;
    }
    __syncthreads();
    for (int64_t e = t; e < total; e += 256) {
        const int32_t v = seg[e];
        if (v >= 0) col[base + e] = v;
    }
}

// A long row by a workgroup of 256 lanes: its candidates (the points of its
// incident cells, the point itself as a filler) sorted by a bitonic network
// in LDS, then one flag per first occurrence and their exclusive sum.  More
// than kLongCap candidates: *err |= 2 (the stencil is not built).  The
// workgroups loop over the long rows (their number is only known on the
// device).
template <int K, bool WRITE>
__global__ void __launch_bounds__(256) long_rows(const int32_t* __restrict__ cells, const int32_t* __restrict__ inc,
                                                 const uint32_t* __restrict__ off, const uint32_t* __restrict__ capp,
                                                 const uint32_t* __restrict__ longs,
                                                 const uint32_t* __restrict__ n_long, uint32_t* __restrict__ deg,
                                                 const int64_t* __restrict__ row_ptr, int32_t* __restrict__ col,
                                                 int* __restrict__ err)
{
    constexpr int kT = 256, kPer = kLongCap / kT;
    constexpr int32_t kFill = INT32_MAX;
    __shared__ int32_t s[kLongCap];
    __shared__ uint32_t part[kT];
    const int t = (int)threadIdx.x;
    const uint32_t nl = *n_long;
    for (uint32_t li = blockIdx.x; li < nl; li += gridDim.x) {
        const int64_t r = longs[li];
        const IncRange ir = inc_range(off, *capp, r);
        const uint32_t p0 = ir.p0, m = (ir.p1 - p0) * K;
        if (m > (uint32_t)kLongCap) {
            if (t == 0) atomicOr(err, 2);
            continue;
        }
        int p2 = 1;
        while (p2 < (int)m) p2 <<= 1;
        for (int i = t; i < p2; i += kT) {
            int32_t u = kFill;
            if (i < (int)m) {
                u = cells[(int64_t)inc[p0 + i / K] * K + i % K];
                if (u == (int32_t)r) u = kFill;
            }
            s[i] = u;
        }
        __syncthreads();
        for (int size = 2; size <= p2; size <<= 1)
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int i = t; i < p2; i += kT) {
                    const int j = i ^ stride;
                    if (j > i) {
                        const bool up = (i & size) == 0;
                        const int32_t a = s[i], b = s[j];
                        if ((a > b) == up) {
                            s[i] = b;
                            s[j] = a;
                        }
                    }
                }
                __syncthreads();
            }
        // lane t owns entries [t kPer, (t + 1) kPer): first occurrences, then their exclusive sum
        uint32_t c = 0;
        for (int k = 0; k < kPer; ++k) {
            const int i = t * kPer + k;
            c += (i < p2 && s[i] != kFill && (i == 0 || s[i] != s[i - 1])) ? 1u : 0u;
        }
        const uint32_t incl = block_inclusive_scan<uint32_t>(c, part, t, kT);
        if constexpr (!WRITE) {
            if (t == kT - 1) deg[r] = incl;
        } else {
            int32_t* out = col + row_ptr[r] + (incl - c);
            for (int k = 0; k < kPer; ++k) {
                const int i = t * kPer + k;
                if (i < p2 && s[i] != kFill && (i == 0 || s[i] != s[i - 1])) *out++ = s[i];
            }
        }
        __syncthreads();
    }
}

constexpr int kLongGrid = 256;

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// Length of the fixed incidence lists, 0 where n of them would not be
// addressable with 32-bit positions (then only packed lists are built).
uint32_t inc_cap(int dim, int64_t n)
{
    const uint32_t cap = dim == 2 ? kIncCap2 : kIncCap3;
    return (uint64_t)n * cap <= 0xffffffffull ? cap : 0u;
}

// Workspace of ring1_build, carved in this order (carve_ring1): incidence
// counts and offsets (n + 1), cursors (n), incidence lists (the larger of
// K n_cells packed and n fixed lists), distinct counts (n + 1), long rows
// (n), stored lists (kRowCap n), scan partial sums, then the error flags,
// the long-row count, the fixed list length in use (0: packed lists) and a copy
// of the entry count.
struct Ring1Work {
    uint32_t *cnt, *cur, *deg, *longs, *n_long, *cap;
    int32_t *inc, *store;
    void* partial;
    int* err;
};

Ring1Work carve_ring1(void* workspace, int dim, int64_t n, int64_t n_cells, size_t* bytes)
{
    const int K = dim + 1;
    const int64_t tiles = (n + 1 + kScanTile - 1) / kScanTile + 1;
    unsigned char* base = static_cast<unsigned char*>(workspace);
    size_t at = 0;
    auto carve = [&](size_t b) {
        void* p = base ? base + at : nullptr;
        at += align256(b);
        return p;
    };
    Ring1Work w;
    w.cnt = static_cast<uint32_t*>(carve(4 * (size_t)(n + 1)));
    w.cur = static_cast<uint32_t*>(carve(4 * (size_t)n));
    w.inc = static_cast<int32_t*>(carve(4 * std::max((size_t)K * n_cells, (size_t)n * inc_cap(dim, n))));
    w.deg = static_cast<uint32_t*>(carve(4 * (size_t)(n + 1)));
    w.longs = static_cast<uint32_t*>(carve(4 * (size_t)n));
    w.store = static_cast<int32_t*>(carve(4 * (size_t)kRowCap * n));
    w.partial = carve(8 * (size_t)tiles);
    w.err = static_cast<int*>(carve(256));
    w.n_long = w.err ? reinterpret_cast<uint32_t*>(w.err + 1) : nullptr;
    w.cap = w.err ? reinterpret_cast<uint32_t*>(w.err + 2) : nullptr;
    if (bytes) *bytes = at;
    return w;
}

}  // namespace

size_t ring1_workspace_bytes(int dim, int64_t n, int64_t n_cells)
{
    size_t bytes = 0;
    (void)carve_ring1(nullptr, dim, n, n_cells, &bytes);
    return bytes;
}


hipError_t ring1_build(int dim, const int32_t* cells, int64_t n_cells, int64_t n, void* workspace, int64_t* row_ptr,
                       int32_t* col, int64_t col_capacity, int64_t* nnz, int* bad_mesh, int* too_long,
                       bool* any_long, hipStream_t stream)
{
    const Ring1Work w = carve_ring1(workspace, dim, n, n_cells, nullptr);
    uint32_t* cnt = w.cnt;
    uint32_t* cur = w.cur;
    int32_t* inc = w.inc;
    uint32_t* deg = w.deg;
    uint32_t* longs = w.longs;
    void* partial = w.partial;
    int* err = w.err;
    uint32_t* n_long = w.n_long;
    // what the host needs at the end, as it lies in the workspace
    struct {
        int flags;
        uint32_t n_long, cap, pad;
        int64_t total;
    } end{};
    static_assert(sizeof(end) == 24, "the counters' layout");
    int64_t* total = reinterpret_cast<int64_t*>(err + 4);
    hipError_t e;
#define FTLE_CHECK(x)                          \
    if ((e = (x)) != hipSuccess) return e;
    FTLE_CHECK(hipMemsetAsync(cnt, 0, 4 * (size_t)(n + 1), stream));
    FTLE_CHECK(hipMemsetAsync(err, 0, 24, stream));
    const dim3 ag(blocks_for(n_cells, kAggThreads * kAggCells)), ab(kAggThreads);
    // 1. fixed lists (with the counts), or the counts alone
    const uint32_t cap = n_cells > 0 ? inc_cap(dim, n) : 0u;
    if (n_cells > 0) {
        if (cap) {
            if (dim == 2)
                hipLaunchKernelGGL((incidence_pass<3, kFixed>), ag, ab, 0, stream, cells, n_cells, n, cnt, inc, err, cap);
            else
                hipLaunchKernelGGL((incidence_pass<4, kFixed>), ag, ab, 0, stream, cells, n_cells, n, cnt, inc, err, cap);
        } else {
            if (dim == 2)
                hipLaunchKernelGGL((incidence_pass<3, kCount>), ag, ab, 0, stream, cells, n_cells, n, cnt, nullptr, err, 0u);
            else
                hipLaunchKernelGGL((incidence_pass<4, kCount>), ag, ab, 0, stream, cells, n_cells, n, cnt, nullptr, err, 0u);
        }
        FTLE_CHECK(hipGetLastError());
    }
    FTLE_CHECK(hipMemcpyAsync(&end.flags, err, sizeof(int), hipMemcpyDeviceToHost, stream));
    FTLE_CHECK(hipStreamSynchronize(stream));
    if (end.flags & 1) {
        *bad_mesh = 1;
        return hipSuccess;
    }
    if (cap && !(end.flags & 4)) {
        // every list fits: the rows read them in place
        FTLE_CHECK(hipMemsetD32Async(reinterpret_cast<hipDeviceptr_t>(w.cap), (int)cap, 1, stream));
    } else if (n_cells > 0) {
        // packed lists: 2. offsets from the counts (cnt becomes off, in place:
        // the tile scan reads a value before writing it), 3. the second pass
        FTLE_CHECK(hipMemsetAsync(err, 0, sizeof(int), stream));
        FTLE_CHECK(exclusive_scan<uint32_t>(cnt, n, cnt, static_cast<uint32_t*>(partial), stream));
        FTLE_CHECK(hipMemcpyAsync(cur, cnt, 4 * (size_t)n, hipMemcpyDeviceToDevice, stream));
        if (dim == 2)
            hipLaunchKernelGGL((incidence_pass<3, kPacked>), ag, ab, 0, stream, cells, n_cells, n, cur, inc, nullptr, 0u);
        else
            hipLaunchKernelGGL((incidence_pass<4, kPacked>), ag, ab, 0, stream, cells, n_cells, n, cur, inc, nullptr, 0u);
        FTLE_CHECK(hipGetLastError());
    }
    // 4. distinct counts, their offsets, then the lists
    const dim3 rg(blocks_for(n, kRowThreads)), rb(kRowThreads);
    if (dim == 2) {
        hipLaunchKernelGGL((ring_rows<3>), rg, rb, 0, stream, cells, inc, cnt, w.cap, n, deg, w.store, longs, n_long);
        hipLaunchKernelGGL((long_rows<3, false>), dim3(kLongGrid), dim3(256), 0, stream, cells, inc, cnt, w.cap, longs,
                           n_long, deg, nullptr, nullptr, err);
    } else {
        hipLaunchKernelGGL((ring_rows<4>), rg, rb, 0, stream, cells, inc, cnt, w.cap, n, deg, w.store, longs, n_long);
        hipLaunchKernelGGL((long_rows<4, false>), dim3(kLongGrid), dim3(256), 0, stream, cells, inc, cnt, w.cap, longs,
                           n_long, deg, nullptr, nullptr, err);
    }
    FTLE_CHECK(hipGetLastError());
    FTLE_CHECK(exclusive_scan<int64_t>(deg, n, row_ptr, static_cast<int64_t*>(partial), stream, total));
    // one copy of flags, long rows and total, and no long-row write where there
    // are none: 1023 x 769 points 162 -> 152 us (a single wait, with the rows
    // queued behind the lists and skipped on an error, gained 2 us and cost 25
    // where a point's cells outgrow the fixed lists)
    FTLE_CHECK(hipMemcpyAsync(&end, err, sizeof end, hipMemcpyDeviceToHost, stream));
    FTLE_CHECK(hipStreamSynchronize(stream));
    *nnz = end.total;
    *any_long = end.n_long != 0;
    if (end.flags & 2) {
        *too_long = 1;
        return hipSuccess;
    }
    if (!col || end.total > col_capacity || end.total == 0) return hipSuccess;
    return ring1_write(dim, cells, n_cells, n, workspace, row_ptr, col, *any_long, stream);
#undef FTLE_CHECK
}

hipError_t ring1_write(int dim, const int32_t* cells, int64_t n_cells, int64_t n, void* workspace,
                       const int64_t* row_ptr, int32_t* col, bool any_long, hipStream_t stream)
{
    const Ring1Work w = carve_ring1(workspace, dim, n, n_cells, nullptr);
    hipLaunchKernelGGL(copy_rows, dim3(blocks_for(n)), dim3(256), 0, stream, w.store, n, w.deg, row_ptr, col);
    if (!any_long) return hipGetLastError();
    if (dim == 2)
        hipLaunchKernelGGL((long_rows<3, true>), dim3(kLongGrid), dim3(256), 0, stream, cells, w.inc, w.cnt, w.cap, w.longs,
                           w.n_long, w.deg, row_ptr, col, w.err);
    else
        hipLaunchKernelGGL((long_rows<4, true>), dim3(kLongGrid), dim3(256), 0, stream, cells, w.inc, w.cnt, w.cap, w.longs,
                           w.n_long, w.deg, row_ptr, col, w.err);
    return hipGetLastError();
}

hipError_t scan_exclusive_u32(const uint32_t* in, int64_t m, uint32_t* out, uint32_t* partial, hipStream_t stream)
{
    return exclusive_scan<uint32_t>(in, m, out, partial, stream);
}

hipError_t scan_exclusive_to_i64(const uint32_t* in, int64_t m, int64_t* out, int64_t* partial, hipStream_t stream)
{
    return exclusive_scan<int64_t>(in, m, out, partial, stream);
}

size_t scan_partial_bytes(int64_t m) { return 8 * (size_t)((m + kScanTile - 1) / kScanTile + 1); }

}  // namespace ftle
