// The whole mesh build on the GPU (ftle_create_mesh_device and
// ftle_create_mesh_device_from_csr): the Morton order of the points, the
// stencil over Morton positions (the one-ring stencil from the cells, the
// axis stencil from it, or a caller's list moved to Morton positions), its
// transpose when it is not symmetric, the tile cut and the compressed tile
// records, and (3D) the inverse normal matrices.  The host-side builder in ftle_host.cpp
// does the same on the CPU, following Section 2.2 (neighbours determined
// once, before the FTLE kernels); the Conclusions name moving that step to
// the accelerator as future work.  Every kernel here reproduces the host's
// result exactly (integer work, and float64 arithmetic evaluated in the same
// order without contraction), so that meshes built either way are the same
// byte for byte.
//
//   bbox_partial    per-workgroup bounds of the coordinates (and whether all
//                   are finite)
//   bbox_reduce / count_wraps
//                   their reduction, and the ends of a lattice's rows and planes
//   order_counts    the caller-order axis test, by counts of a sample's steps
//   morton_keys     each point's interleaved code, quantised as the host
//                   quantises it
//   radix_hist / radix_scatter
//                   a stable LSD radix sort of (code, point) pairs, 8 bits a
//                   pass: per-tile digit counts, their scan (digit-major, so
//                   that equal digits keep tile order), then each key's place
//                   from its tile's offset plus its rank among equal digits
//                   before it (wave ballots; waves and rounds in order)
//   check_relabel   cells validated (index range, repeated points) and
//                   renumbered to Morton positions
//   tile_extent     for candidate Morton ranges: halo points and stencil words
//   tile_record     the record of each tile (the layout in ftle_internal.h):
//                   own points and halo in caller order, index runs, rows as
//                   sorted local slots, shift rows; compact_records then moves
//                   the records together
//   normal_inverse  the 3D normal matrix inverse per point (float64)
//   axis_slots / axis_fill
//                   the axis stencil from the one-ring rows, then its CSR
//   csr_in_count / csr_in_fill
//                   a caller's list checked, moved to Morton positions, sorted
//   transpose_count / transpose_fill / sort_rows / csr_compare
//                   the transpose for the adjoint's tiles, and the test
//                   whether it equals the stencil
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "ftle_device_math.h"
#include "ftle_internal.h"

namespace ftle {
namespace {

inline unsigned blocks_of(int64_t m, int per) { return (unsigned)((m + per - 1) / per); }

// ---------------------------------------------------------------------------
// bounds and Morton codes
// ---------------------------------------------------------------------------
template <int D, typename T>
__global__ void __launch_bounds__(256) bbox_partial(const T* __restrict__ x, int64_t n, double* __restrict__ part,
                                                    unsigned long long* __restrict__ first_bad)
{
    __shared__ double slo[D][256], shi[D][256];
    const int t = (int)threadIdx.x;
    double lo[D], hi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        lo[d] = INFINITY;
        hi[d] = -INFINITY;
    }
    int64_t bad = -1;
    for (int64_t i = (int64_t)blockIdx.x * 256 + t; i < n; i += (int64_t)gridDim.x * 256)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double v = (double)x[i * D + d];
            if (!isfinite(v) && bad < 0) bad = i;
            lo[d] = fmin(lo[d], v);
            hi[d] = fmax(hi[d], v);
        }
    if (bad >= 0) atomicMin(first_bad, (unsigned long long)bad);
#pragma unroll
    for (int d = 0; d < D; ++d) {
        slo[d][t] = lo[d];
        shi[d][t] = hi[d];
    }
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if (t < s)
#pragma unroll
            for (int d = 0; d < D; ++d) {
                slo[d][t] = fmin(slo[d][t], slo[d][t + s]);
                shi[d][t] = fmax(shi[d][t], shi[d][t + s]);
            }
        __syncthreads();
    }
    if (t == 0)
#pragma unroll
        for (int d = 0; d < D; ++d) {
            part[blockIdx.x * 2 * D + d] = slo[d][0];
            part[blockIdx.x * 2 * D + D + d] = shi[d][0];
        }
}

// The caller-order axis test of the host build (the median step between
// consecutive caller points, over sample pairs k stride, k stride + 1, in units
// of the mean spacing: within [0.5, 2] along one axis, at most 0.25 along the
// others) asks of a median only on which side of three limits it lies, and
// that is a count: the element of rank m / 2 is at most t exactly when more
// than m / 2 elements are.  counts[3 d + {0, 1, 2}]: steps along axis d at most
// 0.25, below 0.5, at most 2.  (The pairs' download and the host's selection
// took 0.85 ms of a build, this 7 us.)
template <int D, typename T>
__global__ void __launch_bounds__(256) order_counts(const T* __restrict__ x, int64_t m, int64_t stride,
                                                    MortonParams mp, uint32_t* __restrict__ counts)
{
    __shared__ uint32_t c[3 * D];
    const int t = (int)threadIdx.x;
    if (t < 3 * D) c[t] = 0;
    __syncthreads();
    const int64_t k = (int64_t)blockIdx.x * 256 + t;
    const int64_t i = k * stride;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double step = k < m ? fabs((double)x[(i + 1) * D + d] - (double)x[i * D + d]) / mp.unit[d] : INFINITY;
        const uint64_t b[3] = {__ballot(step <= 0.25), __ballot(step < 0.5), __ballot(step <= 2.0)};
#pragma unroll
        for (int q = 0; q < 3; ++q)
            if ((t & 63) == 0 && b[q]) atomicAdd(&c[3 * d + q], (uint32_t)__popcll(b[q]));
    }
    __syncthreads();
    if (t < 3 * D && c[t]) atomicAdd(&counts[t], c[t]);
}

// The axis of the caller's order by those counts of m samples, or -1.
template <int D>
__device__ inline int order_axis(const uint32_t* counts, int64_t m)
{
    const int64_t h = m / 2;
    int f = -1;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        bool ok = m > 0 && (int64_t)counts[3 * d + 1] <= h && (int64_t)counts[3 * d + 2] > h;
#pragma unroll
        for (int o = 0; o < D; ++o) ok &= o == d || (int64_t)counts[3 * o] > h;
        if (ok) f = d;   // at most one axis passes
    }
    return f;
}

// The bounds from all workgroups' partial ones (one workgroup).
template <int D>
__global__ void __launch_bounds__(256) bbox_reduce(const double* __restrict__ part, int nblocks,
                                                   double* __restrict__ lohi)
{
    __shared__ double s[2 * D][256];
    const int t = (int)threadIdx.x;
#pragma unroll
    for (int q = 0; q < 2 * D; ++q) {
        double v = q < D ? INFINITY : -INFINITY;
        for (int b = t; b < nblocks; b += 256) {
            const double u = part[(int64_t)b * 2 * D + q];
            v = q < D ? fmin(v, u) : fmax(v, u);
        }
        s[q][t] = v;
    }
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if (t < h)
#pragma unroll
            for (int q = 0; q < 2 * D; ++q) s[q][t] = q < D ? fmin(s[q][t], s[q][t + h]) : fmax(s[q][t], s[q][t + h]);
        __syncthreads();
    }
    if (t < 2 * D) lohi[t] = s[t][0];
}

// The steps i -> i + 1 between consecutive caller points that go back along an
// axis by more than half its span (the ends of a lattice's rows and planes):
// wraps[2 d] their number and wraps[2 d + 1] the sum of their (i + 1)^2, modulo
// 2^64.  One more read of the coordinates: 18 us for 1.45 M points in 3D, where
// the order it finds saves 3 of 6 passes of the sort (34 us each) and 80 us of
// tile records.
template <int D, typename T>
__global__ void __launch_bounds__(256) count_wraps(const T* __restrict__ x, int64_t n, const double* __restrict__ lohi,
                                                   unsigned long long* __restrict__ wraps)
{
    __shared__ unsigned long long c[2 * D];
    const int t = (int)threadIdx.x;
    if (t < 2 * D) c[t] = 0;
    __syncthreads();
    double back[D];
    unsigned long long mine[2 * D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        back[d] = -0.5 * (lohi[D + d] - lohi[d]);
        mine[2 * d] = mine[2 * d + 1] = 0;
    }
    for (int64_t i = (int64_t)blockIdx.x * 256 + t; i + 1 < n; i += (int64_t)gridDim.x * 256)
#pragma unroll
        for (int d = 0; d < D; ++d)
            if ((double)x[(i + 1) * D + d] - (double)x[i * D + d] < back[d]) {
                mine[2 * d] += 1;
                mine[2 * d + 1] += (unsigned long long)(i + 1) * (unsigned long long)(i + 1);
            }
#pragma unroll
    for (int q = 0; q < 2 * D; ++q)
        if (mine[q]) atomicAdd(&c[q], mine[q]);
    __syncthreads();
    if (t < 2 * D && c[t]) atomicAdd(&wraps[t], c[t]);
}

__device__ inline uint64_t spread2(uint64_t v)
{
    v &= 0xffffffffULL;
    v = (v | (v << 16)) & 0x0000ffff0000ffffULL;
    v = (v | (v << 8)) & 0x00ff00ff00ff00ffULL;
    v = (v | (v << 4)) & 0x0f0f0f0f0f0f0f0fULL;
    v = (v | (v << 2)) & 0x3333333333333333ULL;
    v = (v | (v << 1)) & 0x5555555555555555ULL;
    return v;
}

__device__ inline uint64_t spread3(uint64_t v)
{
    v &= 0x1fffffULL;
    v = (v | (v << 32)) & 0x001f00000000ffffULL;
    v = (v | (v << 16)) & 0x001f0000ff0000ffULL;
    v = (v | (v << 8)) & 0x100f00f00f00f00fULL;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v << 2)) & 0x1249249249249249ULL;
    return v;
}

// Codes by `plain` if it is a lattice's, else by the parameters for the
// caller's order axis that the counts of m samples show: plain, or (axis) with
// the other axes moved up.
template <int D, typename T>
__global__ void __launch_bounds__(256) morton_keys(const T* __restrict__ x, int64_t n, MortonParams plain,
                                                   MortonParams axis, const uint32_t* __restrict__ counts, int64_t m,
                                                   uint64_t* __restrict__ key, uint32_t* __restrict__ val)
{
#pragma clang fp contract(off)
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    MortonParams mp = plain;
    if (!plain.size[0]) {
        const int fast = order_axis<D>(counts, m);
        if (fast >= 0) mp = axis;
        mp.fast = fast;
    }
    uint64_t code = 0;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        uint64_t q;
        if (mp.size[0]) {
            q = (uint32_t)i / mp.stride[d] % mp.size[d];
        } else {
            const double t = floor((((double)x[i * D + d] - mp.lo[d]) / mp.unit[d] + 0.2) * mp.scale);
            q = (uint64_t)fmin(mp.qmax, fmax(0.0, t));
        }
        if (mp.fast >= 0 && d != mp.fast) q <<= mp.shift_bits;
        code |= (D == 2 ? spread2(q) : spread3(q)) << d;
    }
    key[i] = code;
    val[i] = (uint32_t)i;
}

// ---------------------------------------------------------------------------
// stable LSD radix sort, 8 bits a pass, tiles of kRadixTile keys
// ---------------------------------------------------------------------------
constexpr int kRadixThreads = 256, kRadixRounds = 16, kRadixTile = kRadixThreads * kRadixRounds;

// hist[digit * n_tiles + tile] = keys of the tile with that digit
__global__ void __launch_bounds__(kRadixThreads) radix_hist(const uint64_t* __restrict__ key, int64_t n, int shift,
                                                            uint32_t n_tiles, uint32_t* __restrict__ hist)
{
    __shared__ uint32_t h[256];
    const int t = (int)threadIdx.x;
    h[t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
    for (int j = 0; j < kRadixRounds; ++j) {
        const int64_t i = base + j * kRadixThreads + t;
        if (i < n) atomicAdd(&h[(key[i] >> shift) & 255], 1u);
    }
    __syncthreads();
    hist[(int64_t)t * n_tiles + blockIdx.x] = h[t];
}

// keys of the tile in index order, a round of 256 at a time: the place of a
// key is its digit's offset for the tile, plus the tile's earlier keys of
// that digit, plus those of earlier waves of the round, plus its rank in its
// wave (lanes below it with the same digit, from ballots bit by bit)
__global__ void __launch_bounds__(kRadixThreads) radix_scatter(const uint64_t* __restrict__ key,
                                                               const uint32_t* __restrict__ val, int64_t n, int shift,
                                                               uint32_t n_tiles, const uint32_t* __restrict__ off,
                                                               uint64_t* __restrict__ key2, uint32_t* __restrict__ val2)
{
    constexpr int kWaves = kRadixThreads / 64;
    __shared__ uint32_t run[256];
    __shared__ uint32_t wcnt[kWaves][256];
    const int t = (int)threadIdx.x, lane = t & 63, wave = t >> 6;
    run[t] = off[(int64_t)t * n_tiles + blockIdx.x];
    for (int w = 0; w < kWaves; ++w) wcnt[w][t] = 0;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kRadixTile;
    const uint64_t below = (1ull << lane) - 1;
    for (int j = 0; j < kRadixRounds; ++j) {
        const int64_t i = base + j * kRadixThreads + t;
        const bool live = i < n;
        const uint64_t k = live ? key[i] : 0;
        const uint32_t d = (uint32_t)(k >> shift) & 255u;
        uint64_t same = __ballot(live);
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const bool bit = (d >> b) & 1u;
            const uint64_t m = __ballot(bit);
            same &= bit ? m : ~m;
        }
        if (!live) same = 0;
        const uint32_t rank = (uint32_t)__popcll(same & below);
        if (live && rank == 0) wcnt[wave][d] = (uint32_t)__popcll(same);
        __syncthreads();
        if (live) {
            uint32_t before = run[d];
            for (int w = 0; w < wave; ++w) before += wcnt[w][d];
            const uint32_t p = before + rank;
            key2[p] = k;
            val2[p] = val[i];
        }
        __syncthreads();
        uint32_t add = 0;
        for (int w = 0; w < kWaves; ++w) {
            add += wcnt[w][t];
            wcnt[w][t] = 0;
        }
        run[t] += add;
        __syncthreads();
    }
}

__global__ void __launch_bounds__(256) iota_u32(uint32_t* __restrict__ v, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) v[i] = (uint32_t)i;
}

__global__ void __launch_bounds__(256) invert_perm(const uint32_t* __restrict__ perm, int64_t n,
                                                   int32_t* __restrict__ inv)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r < n) inv[perm[r]] = (int32_t)r;
}

// cells validated (an index outside [0, n): flag 1; a point repeated in a
// cell: flag 2; the lowest such cell in *first) and renumbered
template <int K>
__global__ void __launch_bounds__(256) check_relabel(const int32_t* __restrict__ cells, int64_t n_cells, int64_t n,
                                                     const int32_t* __restrict__ inv, int32_t* __restrict__ mc,
                                                     int* __restrict__ flag, unsigned long long* __restrict__ first)
{
    const int64_t c = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * 256 + threadIdx.x;
    if (c >= n_cells) return;
    int32_t v[K];
#pragma unroll
    for (int a = 0; a < K; ++a) v[a] = cells[c * K + a];
    int kind = 0;
#pragma unroll
    for (int a = 0; a < K; ++a) {
        if ((uint64_t)(int64_t)v[a] >= (uint64_t)n) kind = 1;
#pragma unroll
        for (int q = 0; q < a; ++q)
            if (kind == 0 && v[q] == v[a]) kind = 2;
    }
    if (kind) {
        atomicOr(flag, kind);
        atomicMin(first, (unsigned long long)c);
        return;
    }
#pragma unroll
    for (int a = 0; a < K; ++a) mc[c * K + a] = inv[v[a]];
}

// ---------------------------------------------------------------------------
// tiles.  Shared by the extents and the records: the halo of Morton range [b, e) (the
// stencil's neighbours outside it), gathered in an LDS hash set of Morton
// positions (open addressing).
// ---------------------------------------------------------------------------
constexpr int kTileThreads = 512, kExtentThreads = 256;
constexpr int kTileWaves = kTileThreads / 64;
constexpr int kHashSlots = 2 * kMaxStaged;   // at most kMaxStaged keys are ever kept
constexpr int kChunk = 8;                    // stencil entries a lane loads at once
constexpr int kRowRegs = 32;                 // row entries a lane sorts in registers (longer rows: the workgroup)

__device__ inline uint32_t tile_hash(int32_t v) { return ((uint32_t)v * 2654435761u) >> 21; }   // 11 bits

// Insert every outside neighbour of rows [b, e); keys[] = -1 before.  Returns
// (to every lane) the number of distinct keys, or kMaxStaged + 1 when more
// would be needed.  hlist gets the keys in insertion order.
template <int THREADS>
__device__ inline int gather_halo(const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col, int64_t b,
                                  int64_t e, int32_t* keys, int32_t* hlist, int* count, int t)
{
    static_assert(kHashSlots == 1 << 11, "tile_hash gives 11 bits");
    for (int64_t r = b + t; r < e; r += THREADS) {
        if (__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) > kMaxStaged) break;
        const int64_t p0 = row_ptr[r], p1 = row_ptr[r + 1];
        // kChunk entries loaded together, then inserted (a load past the row
        // end repeats its last entry, which is then found already inserted)
        for (int64_t p = p0; p < p1; p += kChunk) {
            int32_t cs[kChunk];
#pragma unroll
            for (int q = 0; q < kChunk; ++q) cs[q] = col[min(p + q, p1 - 1)];
#pragma unroll
            for (int q = 0; q < kChunk; ++q) {
                const int32_t c = cs[q];
                if (c >= b && c < e) continue;
                uint32_t h = tile_hash(c);
                for (int probe = 0; probe < kHashSlots; ++probe, h = (h + 1) & (kHashSlots - 1)) {
                    const int32_t k = atomicCAS(&keys[h], -1, c);
                    if (k == -1) {
                        const int at = atomicAdd(count, 1);
                        if (at < kMaxStaged) hlist[at] = c;
                        break;
                    }
                    if (k == c) break;
                }
            }
        }
    }
    __syncthreads();
    const int cnt = *count;
    return cnt > kMaxStaged ? kMaxStaged + 1 : cnt;
}

// For each candidate range: its halo size (kMaxStaged + 1 when over) and its
// stencil words (rows padded to multiples of 3).
__global__ void __launch_bounds__(kExtentThreads) tile_extent(const int64_t* __restrict__ row_ptr,
                                                            const int32_t* __restrict__ col,
                                                            const int64_t* __restrict__ ranges,
                                                            uint32_t* __restrict__ halo_words)
{
    __shared__ int32_t keys[kHashSlots];
    __shared__ int32_t hlist[kMaxStaged];
    __shared__ int count;
    __shared__ unsigned long long words;
    const int t = (int)threadIdx.x;
    const int tb = xcd_tile((int)blockIdx.x, (int)gridDim.x);   // XCD-contiguous ranges
    const int64_t b = ranges[2 * tb], e = ranges[2 * tb + 1];
    for (int i = t; i < kHashSlots; i += kExtentThreads) keys[i] = -1;
    if (t == 0) {
        count = 0;
        words = 0;
    }
    __syncthreads();
    unsigned long long w = 0;
    for (int64_t r = b + t; r < e; r += kExtentThreads) w += (uint64_t)((row_ptr[r + 1] - row_ptr[r] + 2) / 3);
    atomicAdd(&words, w);
    int H = kMaxStaged + 1;
    if (e - b <= kMaxStaged) H = gather_halo<kExtentThreads>(row_ptr, col, b, e, keys, hlist, &count, t);
    __syncthreads();
    if (t == 0) {
        halo_words[2 * tb] = (uint32_t)H;
        halo_words[2 * tb + 1] = (uint32_t)(words > 0xffffffffull ? 0xffffffffull : words);
    }
}

// Block-wide exclusive sum of per-lane values; returns the lane's prefix and
// the total in total.  part: kTileWaves words.
__device__ inline uint32_t block_excl(uint32_t v, uint32_t* part, uint32_t& total, int t)
{
    uint32_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint32_t u = __shfl_up(incl, off);
        if ((t & 63) >= off) incl += u;
    }
    __syncthreads();   // part may still be read from the last call
    if ((t & 63) == 63) part[t >> 6] = incl;
    __syncthreads();
    uint32_t before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < kTileWaves; ++w) {
        const uint32_t u = part[w];
        if (w < (t >> 6)) before += u;
        total += u;
    }
    return before + incl - v;
}

// Bitonic sort of m <= 2 kTileThreads 64-bit keys in s (ascending, in place):
// lane t holds keys t and t + kTileThreads; partners within a wave exchange by
// lane shuffles, without a barrier (39 of the 45 steps of 512 keys), the others
// through s.
__device__ inline void sort_keys(uint64_t* s, int m, int t)
{
    int p2 = 1;
    while (p2 < m) p2 <<= 1;
    uint64_t v[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) v[e] = t + e * kTileThreads < m ? s[t + e * kTileThreads] : ~0ull;
    for (int size = 2; size <= p2; size <<= 1)
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            if (stride == kTileThreads) {   // p2 = 2 kTileThreads: both in this lane, ascending
                if (v[0] > v[1]) {
                    const uint64_t u = v[0];
                    v[0] = v[1];
                    v[1] = u;
                }
                continue;
            }
            if (stride >= 64) {
                __syncthreads();
#pragma unroll
                for (int e = 0; e < 2; ++e)
                    if (t + e * kTileThreads < p2) s[t + e * kTileThreads] = v[e];
                __syncthreads();
            }
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int i = t + e * kTileThreads;
                if (i - (t & 63) >= p2) continue;   // whole waves past the keys
                uint64_t o;
                if (stride >= 64) {
                    o = i < p2 ? s[i ^ stride] : ~0ull;
                } else {
                    const uint32_t lo = __shfl_xor((uint32_t)v[e], stride), hi = __shfl_xor((uint32_t)(v[e] >> 32), stride);
                    o = (uint64_t)hi << 32 | lo;
                }
                const bool keep_min = ((i & stride) == 0) == ((i & size) == 0);
                v[e] = keep_min == (v[e] < o) ? v[e] : o;
            }
        }
    __syncthreads();
#pragma unroll
    for (int e = 0; e < 2; ++e)
        if (t + e * kTileThreads < m) s[t + e * kTileThreads] = v[e];
    __syncthreads();
}

// LDS of tile_record besides its row words.
struct TileScratch {
    int32_t keys[kHashSlots];         // halo hash set (Morton positions)
    uint16_t hslot[kHashSlots];       // their slots
    uint64_t sort[kMaxStaged];        // sort keys; the halo in insertion order before; counters and long rows after
    uint32_t caller[kMaxStaged];      // caller index of each staged slot
    uint16_t own_slot[kMaxStaged];    // slot of own point b + i
    uint16_t woff[kMaxStaged + 8];    // row l's first word
    uint32_t part[kTileWaves];
    uint32_t smask[kMaxStaged / 32], spre[kMaxStaged / 32];                        // per group of 32 slots
    uint32_t mask[kMaxStaged / 32], pre[kMaxStaged / 32], last[kMaxStaged / 32];
    int count, n_long;
};

// The slot of Morton position c in the tile of P points from b.
__device__ inline uint32_t slot_of(const TileScratch& q, int64_t b, int P, int32_t c)
{
    const uint32_t o = (uint32_t)(c - (int32_t)b);
    if (o < (uint32_t)P) return q.own_slot[o];
    uint32_t h = tile_hash(c);
    while (q.keys[h] != c) h = (h + 1) & (kHashSlots - 1);
    return q.hslot[h];
}

// A row of at most N entries (stencil entries col[p0, p0 + len), len > 0) into
// its words, ascending by slot, padded with the row's own slot l.
template <int N>
__device__ inline void short_row(const TileScratch& q, const int32_t* __restrict__ col, int64_t b, int P, int64_t p0,
                                 int len, uint32_t l, uint32_t* out)
{
    uint32_t v[N];
    // a batch of entries' loads together, then the first probe of each (the
    // tables' reads then overlap), then the few that collided
    constexpr int kBatch = N <= 16 ? 16 : 8;   // (registers)
#pragma unroll
    for (int k0 = 0; k0 < N; k0 += kBatch) {
        int32_t c[kBatch];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) c[k] = col[p0 + min(k0 + k, len - 1)];
#pragma unroll
        for (int k = 0; k < kBatch; ++k) {
            const uint32_t o = (uint32_t)(c[k] - (int32_t)b), h = tile_hash(c[k]);
            const bool own = o < (uint32_t)P;
            const int32_t found = q.keys[h];
            uint32_t s = own ? q.own_slot[o] : q.hslot[h];
            if (!own && found != c[k]) s = slot_of(q, b, P, c[k]);
            v[k0 + k] = k0 + k < len ? s : 0xffffu;
        }
    }
    odd_even_sort<0, N>(v);
    const int nw = (len + 2) / 3;
#pragma unroll
    for (int w = 0; w < (N + 2) / 3; ++w) {
        if (w < nw) {
            const uint32_t v1 = 3 * w + 1 < N ? v[3 * w + 1 < N ? 3 * w + 1 : 0] : 0xffffu;
            const uint32_t v2 = 3 * w + 2 < N ? v[3 * w + 2 < N ? 3 * w + 2 : 0] : 0xffffu;
            uint32_t word = v[3 * w] | (3 * w + 1 < len ? v1 : l) << 10 | (3 * w + 2 < len ? v2 : l) << 20;
            if (w == nw - 1) word |= (uint32_t)(3 * nw - len) << 30;
            out[w] = word;
        }
    }
}

// The record of one tile per workgroup, in one pass: written to
// stage + 16 stage_off[t], where the largest record of a tile with these
// points, halo and words has room; its counts go to counts[4 t] = {nw, nr, nx,
// nwf}, and compact_records moves the records to their final places.  The
// rows are kept packed in LDS (dynamic: the largest tile's words), where a row
// that continues the previous one is found by comparing words.
//
// What bounds it is latency, LDS and barriers, not bytes: 512 threads (a row
// each), rows sorted in registers by a network, sorts by lane shuffles, masks by
// ballots and scans by shuffles, and registers and LDS for four workgroups a CU.
// 127 x 113 x 101 points: 260 us and 11 us for the compaction (two passes of 256
// threads with the rows in global memory between them, sorted by insertion in
// LDS, took 409 + 275 us); in 2962 lattice blocks instead of 5502 tiles 178 us
// and 8 us.
__global__ void __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(8)))
tile_record(const int64_t* __restrict__ row_ptr,
                                                            const int32_t* __restrict__ col,
                                                            const uint32_t* __restrict__ perm,
                                                            const int64_t* __restrict__ ranges,
                                                            const uint32_t* __restrict__ stage_off,
                                                            uint32_t* __restrict__ counts,
                                                            unsigned char* __restrict__ stage)
{
    extern __shared__ uint32_t words[];   // row l's words at words[woff[l]]
    __shared__ TileScratch q;
    const int t = (int)threadIdx.x;
    const int tb = xcd_tile((int)blockIdx.x, (int)gridDim.x);   // XCD-contiguous tiles
    const int64_t b = ranges[2 * tb], e = ranges[2 * tb + 1];
    const int P = (int)(e - b);
    for (int i = t; i < kHashSlots; i += kTileThreads) q.keys[i] = -1;
    if (t == 0) {
        q.count = 0;
        q.n_long = 0;
    }
    // own points in caller order
    for (int i = t; i < P; i += kTileThreads) q.sort[i] = ((uint64_t)perm[b + i] << 32) | (uint32_t)i;
    __syncthreads();
    sort_keys(q.sort, P, t);
    for (int l = t; l < P; l += kTileThreads) {
        q.own_slot[q.sort[l] & 0xffffffffu] = (uint16_t)l;
        q.caller[l] = (uint32_t)(q.sort[l] >> 32);
    }
    __syncthreads();
    // the halo in caller order (the extents admitted only tiles with P + H <= kMaxStaged)
    int32_t* hlist = reinterpret_cast<int32_t*>(q.sort);
    const int H = gather_halo<kTileThreads>(row_ptr, col, b, e, q.keys, hlist, &q.count, t);
    if (P + H > kMaxStaged) {
        if (t == 0)
            for (int k = 0; k < 4; ++k) counts[4 * tb + k] = ~0u;
        return;
    }
    {
        uint64_t v[2];
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (t + k * kTileThreads < H) {
                const int32_t c = hlist[t + k * kTileThreads];
                v[k] = (uint64_t)perm[c] << 32 | (uint32_t)c;
            }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 2; ++k)
            if (t + k * kTileThreads < H) q.sort[t + k * kTileThreads] = v[k];
        __syncthreads();
    }
    sort_keys(q.sort, H, t);
    for (int h = t; h < H; h += kTileThreads) {
        const int32_t c = (int32_t)(q.sort[h] & 0xffffffffu);
        q.caller[P + h] = (uint32_t)(q.sort[h] >> 32);
        uint32_t k = tile_hash(c);
        while (q.keys[k] != c) k = (k + 1) & (kHashSlots - 1);
        q.hslot[k] = (uint16_t)(P + h);
    }
    // rows: their words' offsets, in slot order
    for (int i = t; i < P; i += kTileThreads)
        q.woff[q.own_slot[i]] = (uint16_t)((row_ptr[b + i + 1] - row_ptr[b + i] + 2) / 3);
    __syncthreads();
    uint32_t nwf = 0;
    for (int l0 = 0; l0 < P; l0 += kTileThreads) {
        const uint32_t n = l0 + t < P ? q.woff[l0 + t] : 0u;
        uint32_t total;
        const uint32_t o = block_excl(n, q.part, total, t);
        if (l0 + t < P) q.woff[l0 + t] = (uint16_t)(nwf + o);
        nwf += total;
    }
    if (t == 0) q.woff[P] = (uint16_t)nwf;
    __syncthreads();
    // each row by a lane; long ones are listed for the workgroup
    uint32_t* cnt = reinterpret_cast<uint32_t*>(q.sort);   // kMaxStaged counters, then the list
    uint16_t* longs = reinterpret_cast<uint16_t*>(cnt + kMaxStaged);
    static_assert(sizeof(q.sort) >= kMaxStaged * 6, "counters and long rows fit the sort buffer");
    for (int i = t; i < P; i += kTileThreads) {
        const int64_t p0 = row_ptr[b + i];
        const int64_t len = row_ptr[b + i + 1] - p0;
        const uint32_t l = q.own_slot[i];
        uint32_t* out = words + q.woff[l];
        if (len <= 0) continue;
        if (len <= 16) {
            short_row<16>(q, col, b, P, p0, (int)len, l, out);
        } else if (len <= kRowRegs) {
            short_row<kRowRegs>(q, col, b, P, p0, (int)len, l, out);
        } else {
            for (int64_t w = 0; w < (len + 2) / 3; ++w) out[w] = 0;
            longs[atomicAdd(&q.n_long, 1)] = (uint16_t)i;
        }
    }
    __syncthreads();
    // long rows: occurrences counted per slot, then listed in slot order
    for (int k = 0; k < q.n_long; ++k) {
        const int i = longs[k];
        const int64_t p0 = row_ptr[b + i];
        const int len = (int)(row_ptr[b + i + 1] - p0);   // at most 3 nwf
        const uint32_t l = q.own_slot[i];
        uint32_t* out = words + q.woff[l];
        for (int j = t; j < kMaxStaged; j += kTileThreads) cnt[j] = 0;
        __syncthreads();
        for (int j = t; j < len; j += kTileThreads) atomicAdd(&cnt[slot_of(q, b, P, col[p0 + j])], 1u);
        __syncthreads();
        const uint32_t c0 = cnt[2 * t], c1 = cnt[2 * t + 1];
        uint32_t total;
        uint32_t at = block_excl(c0 + c1, q.part, total, t);
        for (uint32_t j = 0; j < c0 + c1; ++j, ++at)
            atomicOr(&out[at / 3], (uint32_t)(2 * t + (j < c0 ? 0 : 1)) << (10 * (at % 3)));
        if (t == 0) {
            const int end = (len + 2) / 3 * 3;
            for (int j = len; j < end; ++j) atomicOr(&out[j / 3], l << (10 * (j % 3)));
            atomicOr(&out[end / 3 - 1], (uint32_t)(end - len) << 30);
        }
        __syncthreads();
    }
    // runs of consecutive caller indices, explicit rows (not the previous row
    // with every slot plus one), as masks and their prefix counts
    const int S = P + H, G = (S + 31) / 32, Q = (P + 31) / 32;
    for (int l0 = 0; l0 < S; l0 += kTileThreads) {
        const int l = l0 + t;
        const uint64_t m = __ballot(l < S && (l == 0 || q.caller[l] != q.caller[l - 1] + 1u));
        if ((t & 31) == 0 && l < S) q.smask[l >> 5] = (t & 32) ? (uint32_t)(m >> 32) : (uint32_t)m;
    }
    __syncthreads();
    if (t < 64) {   // (G and Q are at most 32)
        const uint32_t c = t < G ? (uint32_t)__popc(q.smask[t]) : 0u;
        uint32_t incl = c;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const uint32_t u = __shfl_up(incl, off);
            if (t >= off) incl += u;
        }
        if (t < 32) q.spre[t] = incl - c;
        if (t == 31) q.count = (int)incl;
    }
    __syncthreads();
    const uint32_t nr = (uint32_t)q.count;
    bool expl[2] = {false, false};
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int l = t + k * kTileThreads;
        if (l < P) {
            const uint32_t o = q.woff[l], n = q.woff[l + 1] - o;
            bool shift = l > 0 && o - q.woff[l - 1] == n;
            if (shift) {
                const uint32_t *w0 = words + q.woff[l - 1], *w1 = words + o;
                for (uint32_t j = 0; shift && j < n; ++j) {
                    const uint32_t u = w0[j] & 0x3fffffffu;
                    shift = (w1[j] & 0x3fffffffu) == u + 0x00100401u;
                    // slot 1023 has no successor: its carry must not pass for one
                    if (S == kMaxStaged)
                        shift &= (u & 0x3ffu) != 0x3ffu && (u & 0xffc00u) != 0xffc00u && (u & 0x3ff00000u) != 0x3ff00000u;
                }
            }
            expl[k] = !shift;
        }
        const uint64_t m = __ballot(expl[k]);
        if ((t & 31) == 0 && l < P) q.mask[l >> 5] = (t & 32) ? (uint32_t)(m >> 32) : (uint32_t)m;
    }
    __syncthreads();
    if (t < 64) {
        const uint32_t m = t < Q ? q.mask[t] : 0u, c = (uint32_t)__popc(m);
        uint32_t incl = c, last = m ? 32u * (uint32_t)t + 31u - (uint32_t)__clz((int)m) : 0u;
#pragma unroll
        for (int off = 1; off < 32; off <<= 1) {
            const uint32_t u = __shfl_up(incl, off), v = __shfl_up(last, off);
            if (t >= off) {
                incl += u;
                last = max(last, v);
            }
        }
        const uint32_t before = __shfl_up(last, 1);
        if (t < 32) {
            q.pre[t] = incl - c;
            q.last[t] = t ? before : 0u;   // the last explicit row before group t
        }
        if (t == 31) q.count = (int)incl;
    }
    __syncthreads();
    const uint32_t nx = (uint32_t)q.count;
    uint32_t nw = 0, kw[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int l = t + k * kTileThreads;
        const uint32_t c = expl[k] ? (uint32_t)q.woff[l + 1] - q.woff[l] : 0u;
        uint32_t total;
        kw[k] = nw + block_excl(c, q.part, total, t);
        nw += total;
    }
    const RecLayout R = rec_layout((uint32_t)P, (uint32_t)H, nw, nr, nx);
    unsigned char* out = stage + (size_t)16 * stage_off[tb];
    uint32_t* wd = reinterpret_cast<uint32_t*>(out);
    uint16_t* xend = reinterpret_cast<uint16_t*>(out + R.xend);
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const int l = t + k * kTileThreads;
        if (l < S && (q.smask[l >> 5] >> (l & 31) & 1u))
            reinterpret_cast<uint32_t*>(
                out + R.runs)[q.spre[l >> 5] + (uint32_t)__popc(q.smask[l >> 5] & ((1u << (l & 31)) - 1u))] =
                q.caller[l] - (uint32_t)l;
        if (!expl[k]) continue;
        const uint32_t o = q.woff[l], n = q.woff[l + 1] - o;
        for (uint32_t j = 0; j < n; ++j) wd[kw[k] + j] = words[o + j];
        xend[q.pre[l >> 5] + (uint32_t)__popc(q.mask[l >> 5] & ((1u << (l & 31)) - 1u))] = (uint16_t)(kw[k] + n);
    }
    if (t < G) {
        reinterpret_cast<uint32_t*>(out + R.smask)[t] = q.smask[t];
        reinterpret_cast<uint16_t*>(out + R.spre)[t] = (uint16_t)q.spre[t];
    }
    if (t < Q) {
        reinterpret_cast<uint32_t*>(out + R.xmask)[t] = q.mask[t];
        reinterpret_cast<uint16_t*>(out + R.xpre)[t] = (uint16_t)q.pre[t];
        reinterpret_cast<uint16_t*>(out + R.xlast)[t] = (uint16_t)q.last[t];
    }
    if (t == 0) {
        for (uint32_t at = R.xend + 2u * nx; at < R.bytes; at += 2) *reinterpret_cast<uint16_t*>(out + at) = 0;
        counts[4 * tb] = nw;
        counts[4 * tb + 1] = nr;
        counts[4 * tb + 2] = nx;
        counts[4 * tb + 3] = nwf;
    }
}

// Record t from its place in the stage to 16 meta[t].rec_off.
__global__ void __launch_bounds__(128) compact_records(const uint32_t* __restrict__ stage_off,
                                                       const TileMeta* __restrict__ meta,
                                                       const unsigned char* __restrict__ stage,
                                                       unsigned char* __restrict__ rec)
{
    const TileMeta m = meta[blockIdx.x];
    const uint4* src = reinterpret_cast<const uint4*>(stage) + stage_off[blockIdx.x];
    uint4* dst = reinterpret_cast<uint4*>(rec) + m.rec_off;
    const uint32_t n = rec_layout(m).bytes / 16;
    for (uint32_t i = threadIdx.x; i < n; i += 128) dst[i] = src[i];
}

constexpr int kAhead = 4;   // neighbours of a row loaded together

// The float64 inverse of each point's normal matrix M = sum (x_j - x_i)(x_j - x_i)^T
// over its row (Morton positions), in caller order, NaN where the rank test fails.
// Bound by the chain of a neighbour's position, caller index and coordinates,
// so a row's neighbours go through it kAhead at a time (1.45 M points, 127 ->
// 77 us; eight at a time 77); the sums keep the row's order.
template <typename T>
__global__ void __launch_bounds__(256) normal_inverse(const int64_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ col,
                                                      const uint32_t* __restrict__ perm, const T* __restrict__ x,
                                                      int64_t n, double tau, T* __restrict__ out)
{
#pragma clang fp contract(off)
    const int64_t r = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * 256 + threadIdx.x;
    if (r >= n) return;
    const int64_t i = perm[r];
    const double xi0 = (double)x[i * 3], xi1 = (double)x[i * 3 + 1], xi2 = (double)x[i * 3 + 2];
    double m00 = 0, m01 = 0, m02 = 0, m11 = 0, m12 = 0, m22 = 0;
    const int64_t p1 = row_ptr[r + 1];
    for (int64_t p = row_ptr[r]; p < p1; p += kAhead) {
        int64_t j[kAhead];
        T v[kAhead][3];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) j[u] = p + u < p1 ? col[p + u] : r;   // past the row: no difference, adds +0
#pragma unroll
        for (int u = 0; u < kAhead; ++u) j[u] = perm[j[u]];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int d = 0; d < 3; ++d) v[u][d] = x[j[u] * 3 + d];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const double d0 = (double)v[u][0] - xi0, d1 = (double)v[u][1] - xi1, d2 = (double)v[u][2] - xi2;
            m00 += d0 * d0;
            m01 += d0 * d1;
            m02 += d0 * d2;
            m11 += d1 * d1;
            m12 += d1 * d2;
            m22 += d2 * d2;
        }
    }
    const double a00 = m11 * m22 - m12 * m12, a01 = m02 * m12 - m01 * m22, a02 = m01 * m12 - m02 * m11;
    const double a11 = m00 * m22 - m02 * m02, a12 = m01 * m02 - m00 * m12, a22 = m00 * m11 - m01 * m01;
    const double det = m00 * a00 + m01 * a01 + m02 * a02;
    const double tr3 = (m00 + m11 + m22) / 3.0;
    double v[6] = {a00 / det, a01 / det, a02 / det, a11 / det, a12 / det, a22 / det};
    if (!(det > tau * tr3 * tr3 * tr3))
        for (double& q : v) q = __builtin_nan("");
#pragma unroll
    for (int k = 0; k < 6; ++k) out[i * 6 + k] = (T)v[k];
}

// ---------------------------------------------------------------------------
// The axis stencil over Morton positions (FTLE_STENCIL_AXIS), as the host
// builds it: per signed axis direction the one-ring neighbour on that side
// with the largest cosine to the axis (float64, no contraction, ties to the
// smaller caller index), in slot order (-x, +x, -y, +y[, -z, +z]), absent
// sides dropped, a neighbour chosen twice listed twice.
// ---------------------------------------------------------------------------
template <int D, typename T>
__global__ void __launch_bounds__(256) axis_slots(const T* __restrict__ x, const uint32_t* __restrict__ perm,
                                                  const int64_t* __restrict__ row_ptr, const int32_t* __restrict__ col,
                                                  int64_t n, int32_t* __restrict__ slots, uint32_t* __restrict__ cnt)
{
#pragma clang fp contract(off)
    const int64_t r = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * 256 + threadIdx.x;
    if (r >= n) return;
    const int64_t i = perm[r];
    double xi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) xi[d] = (double)x[i * D + d];
    int32_t best[2 * D];
    uint32_t best_u[2 * D];
    double best_c[2 * D];
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
        best[k] = -1;
        best_u[k] = 0;
        best_c[k] = 0.0;
    }
    const int64_t p1 = row_ptr[r + 1];
    for (int64_t p = row_ptr[r]; p < p1; p += kAhead) {
        int32_t c[kAhead];
        uint32_t j[kAhead];
        T v[kAhead][D];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) c[u] = p + u < p1 ? col[p + u] : (int32_t)r;   // past the row: on no side
#pragma unroll
        for (int u = 0; u < kAhead; ++u) j[u] = perm[c[u]];
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
#pragma unroll
            for (int d = 0; d < D; ++d) v[u][d] = x[(int64_t)j[u] * D + d];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            double dx[D];
            double nrm2 = 0.0;
#pragma unroll
            for (int d = 0; d < D; ++d) {
                dx[d] = (double)v[u][d] - xi[d];
                nrm2 = nrm2 + dx[d] * dx[d];
            }
            const double nrm = sqrt(nrm2);
#pragma unroll
            for (int d = 0; d < D; ++d) {
                if (dx[d] == 0.0) continue;            // on no side (whole waves on a lattice)
                const double cs = fabs(dx[d]) / nrm;   // one division for both sides
#pragma unroll
                for (int sg = 0; sg < 2; ++sg) {
                    const int k = 2 * d + sg;
                    const bool take = (sg ? dx[d] : -dx[d]) > 0.0 &&
                                      (best[k] < 0 || cs > best_c[k] || (cs == best_c[k] && j[u] < best_u[k]));
                    best_c[k] = take ? cs : best_c[k];
                    best[k] = take ? c[u] : best[k];
                    best_u[k] = take ? j[u] : best_u[k];
                }
            }
        }
    }
    uint32_t m = 0;
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
        slots[r * 2 * D + k] = best[k];
        m += best[k] >= 0 ? 1u : 0u;
    }
    cnt[r] = m;
}

template <int D>
__global__ void __launch_bounds__(256) axis_fill(const int32_t* __restrict__ slots, const int64_t* __restrict__ row_ptr,
                                                 int64_t n, int32_t* __restrict__ col)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    int64_t q = row_ptr[r];
#pragma unroll
    for (int k = 0; k < 2 * D; ++k) {
        const int32_t c = slots[r * 2 * D + k];
        if (c >= 0) col[q++] = c;
    }
}

// Transpose of a CSR over Morton positions: column counts, then (after their
// scan) each entry placed by an atomic cursor, then each row sorted (rows
// ascend, as the host's counting transpose leaves them).
__global__ void __launch_bounds__(256) transpose_count(const int32_t* __restrict__ col, int64_t nnz,
                                                       uint32_t* __restrict__ tcnt)
{
    const int64_t p = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (p < nnz) atomicAdd(&tcnt[col[p]], 1u);
}

__global__ void __launch_bounds__(256) transpose_fill(const int64_t* __restrict__ row_ptr,
                                                      const int32_t* __restrict__ col, int64_t n,
                                                      const int64_t* __restrict__ trp, uint32_t* __restrict__ cur,
                                                      int32_t* __restrict__ tcol)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    for (int64_t p = row_ptr[r]; p < row_ptr[r + 1]; ++p) {
        const int32_t c = col[p];
        tcol[trp[c] + atomicAdd(&cur[c], 1u)] = (int32_t)r;
    }
}

__global__ void __launch_bounds__(256) sort_rows(const int64_t* __restrict__ row_ptr, int64_t n,
                                                 int32_t* __restrict__ col)
{
    const int64_t r = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (r >= n) return;
    int32_t* row = col + row_ptr[r];
    const int64_t len = row_ptr[r + 1] - row_ptr[r];
    for (int64_t a = 1; a < len; ++a) {
        const int32_t v = row[a];
        int64_t k = a;
        while (k > 0 && row[k - 1] > v) {
            row[k] = row[k - 1];
            --k;
        }
        row[k] = v;
    }
}

// *differ = 1 where two CSRs of n rows and nnz entries differ
__global__ void __launch_bounds__(256) csr_compare(const int64_t* __restrict__ rp_a, const int32_t* __restrict__ col_a,
                                                   const int64_t* __restrict__ rp_b, const int32_t* __restrict__ col_b,
                                                   int64_t n, int64_t nnz, int* __restrict__ differ)
{
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if ((i <= n && rp_a[i] != rp_b[i]) || (i < nnz && col_a[i] != col_b[i])) *differ = 1;
}

// ---------------------------------------------------------------------------
// A caller's CSR over caller indices moved to Morton positions: per Morton
// row r (caller row perm[r]) the entries that are neither -1 nor the point
// itself, renumbered and sorted ascending (repeats kept).  The count pass also
// checks the input: err[0] lowers to 0 for row_ptr[0] != 0 and to i + 1 for a
// row i whose end precedes its start; err[1] lowers to the position of an
// entry outside [-1, n).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) csr_in_count(const int64_t* __restrict__ row_ptr,
                                                    const int32_t* __restrict__ col, int64_t n, int64_t nnz_in,
                                                    const uint32_t* __restrict__ perm, uint32_t* __restrict__ cnt,
                                                    unsigned long long* __restrict__ err)
{
    const int64_t r = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * 256 + threadIdx.x;
    if (r >= n) return;
    if (r == 0 && row_ptr[0] != 0) atomicMin(&err[0], 0ull);
    const int64_t i = perm[r];
    const int64_t p0 = row_ptr[i], p1 = row_ptr[i + 1];
    uint32_t c = 0;
    if (p1 < p0) {
        atomicMin(&err[0], (unsigned long long)(i + 1));
    } else if (p0 >= 0 && p1 <= nnz_in) {
        for (int64_t p = p0; p < p1; ++p) {
            const int32_t v = col[p];
            if (v < -1 || v >= n)
                atomicMin(&err[1], (unsigned long long)p);
            else if (v >= 0 && v != (int32_t)i)
                ++c;
        }
    }
    cnt[r] = c;
}

__global__ void __launch_bounds__(256) csr_in_fill(const int64_t* __restrict__ row_ptr,
                                                   const int32_t* __restrict__ col, int64_t n,
                                                   const uint32_t* __restrict__ perm, const int32_t* __restrict__ inv,
                                                   const int64_t* __restrict__ out_rp, int32_t* __restrict__ out)
{
    const int64_t r = (int64_t)xcd_tile((int)blockIdx.x, (int)gridDim.x) * 256 + threadIdx.x;
    if (r >= n) return;
    const int64_t i = perm[r];
    int32_t* row = out + out_rp[r];
    int64_t len = 0;
    for (int64_t p = row_ptr[i]; p < row_ptr[i + 1]; ++p) {
        const int32_t v = col[p];
        if (v < 0 || v == (int32_t)i) continue;
        const int32_t u = inv[v];
        int64_t k = len;
        while (k > 0 && row[k - 1] > u) {
            row[k] = row[k - 1];
            --k;
        }
        row[k] = u;
        ++len;
    }
}

}  // namespace

// ---------------------------------------------------------------------------
// launchers (ftle_internal.h)
// ---------------------------------------------------------------------------
hipError_t mb_bbox(int dim, bool f64, const void* x, int64_t n, double* part, int nblocks,
                   unsigned long long* first_bad, hipStream_t s)
{
#define FTLE_MB(D, T) hipLaunchKernelGGL((bbox_partial<D, T>), dim3(nblocks), dim3(256), 0, s, static_cast<const T*>(x), n, part, first_bad)
    if (dim == 2) {
        if (f64) FTLE_MB(2, double); else FTLE_MB(2, float);
    } else {
        if (f64) FTLE_MB(3, double); else FTLE_MB(3, float);
    }
#undef FTLE_MB
    return hipGetLastError();
}

hipError_t mb_wraps(int dim, bool f64, const void* x, int64_t n, const double* part, int nblocks, double* lohi,
                    unsigned long long* wraps, hipStream_t s)
{
    if (dim == 2)
        hipLaunchKernelGGL(bbox_reduce<2>, dim3(1), dim3(256), 0, s, part, nblocks, lohi);
    else
        hipLaunchKernelGGL(bbox_reduce<3>, dim3(1), dim3(256), 0, s, part, nblocks, lohi);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
#define FTLE_MB(D, T) hipLaunchKernelGGL((count_wraps<D, T>), dim3(nblocks), dim3(256), 0, s, static_cast<const T*>(x), n, lohi, wraps)
    if (dim == 2) {
        if (f64) FTLE_MB(2, double); else FTLE_MB(2, float);
    } else {
        if (f64) FTLE_MB(3, double); else FTLE_MB(3, float);
    }
#undef FTLE_MB
    return hipGetLastError();
}

hipError_t mb_order_counts(int dim, bool f64, const void* x, int64_t m, int64_t stride, const MortonParams& mp,
                           uint32_t* counts, hipStream_t s)
{
    if (m <= 0) return hipSuccess;
#define FTLE_MB(D, T) hipLaunchKernelGGL((order_counts<D, T>), dim3(blocks_of(m, 256)), dim3(256), 0, s, static_cast<const T*>(x), m, stride, mp, counts)
    if (dim == 2) {
        if (f64) FTLE_MB(2, double); else FTLE_MB(2, float);
    } else {
        if (f64) FTLE_MB(3, double); else FTLE_MB(3, float);
    }
#undef FTLE_MB
    return hipGetLastError();
}

hipError_t mb_morton(int dim, bool f64, const void* x, int64_t n, const MortonParams& plain, const MortonParams& axis,
                     const uint32_t* counts, int64_t m, uint64_t* key, uint32_t* val, hipStream_t s)
{
#define FTLE_MB(D, T) hipLaunchKernelGGL((morton_keys<D, T>), dim3(blocks_of(n, 256)), dim3(256), 0, s, static_cast<const T*>(x), n, plain, axis, counts, m, key, val)
    if (dim == 2) {
        if (f64) FTLE_MB(2, double); else FTLE_MB(2, float);
    } else {
        if (f64) FTLE_MB(3, double); else FTLE_MB(3, float);
    }
#undef FTLE_MB
    return hipGetLastError();
}

size_t mb_sort_scratch_bytes(int64_t n)
{
    const int64_t tiles = (n + kRadixTile - 1) / kRadixTile;
    const size_t h = (size_t)256 * tiles + 1;
    return 8 * (size_t)n + 4 * (size_t)n + ((4 * h + 255) & ~(size_t)255) + scan_partial_bytes((int64_t)h) + 256;
}

hipError_t mb_sort(uint64_t* key, uint32_t* val, int64_t n, int key_bits, void* scratch, uint32_t** sorted_val,
                   hipStream_t s)
{
    unsigned char* w = static_cast<unsigned char*>(scratch);
    uint64_t* key2 = reinterpret_cast<uint64_t*>(w);
    uint32_t* val2 = reinterpret_cast<uint32_t*>(w + 8 * (size_t)n);
    const int64_t tiles = (n + kRadixTile - 1) / kRadixTile;
    const int64_t h = 256 * tiles;
    uint32_t* hist = reinterpret_cast<uint32_t*>(w + 12 * (size_t)n);
    uint32_t* partial = reinterpret_cast<uint32_t*>(w + 12 * (size_t)n + ((4 * (size_t)(h + 1) + 255) & ~(size_t)255));
    hipError_t e;
    for (int shift = 0; shift < key_bits; shift += 8) {
        hipLaunchKernelGGL(radix_hist, dim3((unsigned)tiles), dim3(kRadixThreads), 0, s, key, n, shift,
                           (uint32_t)tiles, hist);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = scan_exclusive_u32(hist, h, hist, partial, s)) != hipSuccess) return e;
        hipLaunchKernelGGL(radix_scatter, dim3((unsigned)tiles), dim3(kRadixThreads), 0, s, key, val, n, shift,
                           (uint32_t)tiles, hist, key2, val2);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        std::swap(key, key2);
        std::swap(val, val2);
    }
    *sorted_val = val;
    return hipSuccess;
}

hipError_t mb_iota(uint32_t* v, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(iota_u32, dim3(blocks_of(n, 256)), dim3(256), 0, s, v, n);
    return hipGetLastError();
}

hipError_t mb_invert(const uint32_t* perm, int64_t n, int32_t* inv, hipStream_t s)
{
    hipLaunchKernelGGL(invert_perm, dim3(blocks_of(n, 256)), dim3(256), 0, s, perm, n, inv);
    return hipGetLastError();
}

hipError_t mb_relabel(int dim, const int32_t* cells, int64_t n_cells, int64_t n, const int32_t* inv, int32_t* mc,
                      int* flag, unsigned long long* first, hipStream_t s)
{
    if (n_cells == 0) return hipSuccess;
    if (dim == 2)
        hipLaunchKernelGGL(check_relabel<3>, dim3(blocks_of(n_cells, 256)), dim3(256), 0, s, cells, n_cells, n, inv, mc,
                           flag, first);
    else
        hipLaunchKernelGGL(check_relabel<4>, dim3(blocks_of(n_cells, 256)), dim3(256), 0, s, cells, n_cells, n, inv, mc,
                           flag, first);
    return hipGetLastError();
}

hipError_t mb_tile_extent(const int64_t* row_ptr, const int32_t* col, const int64_t* ranges, int64_t n_ranges,
                          uint32_t* halo_words, hipStream_t s)
{
    if (n_ranges == 0) return hipSuccess;
    hipLaunchKernelGGL(tile_extent, dim3((unsigned)n_ranges), dim3(kExtentThreads), 0, s, row_ptr, col, ranges,
                       halo_words);
    return hipGetLastError();
}

hipError_t mb_tile_record(const int64_t* row_ptr, const int32_t* col, const uint32_t* perm, const int64_t* ranges,
                          int64_t n_tiles, uint32_t max_words, const uint32_t* stage_off, uint32_t* counts,
                          unsigned char* stage, hipStream_t s)
{
    if (n_tiles == 0) return hipSuccess;
    // The largest tile's words for every tile: a few long rows anywhere take
    // workgroups from each CU (30 rows of 899 among 10^6 points: 0.09 -> 0.40 ms,
    // the long rows' own work included, of a build of 12.1 ms).
    const size_t lds = 4 * (size_t)max_words;
    const hipError_t e = allow_lds(reinterpret_cast<const void*>(&tile_record), sizeof(TileScratch) + lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(tile_record, dim3((unsigned)n_tiles), dim3(kTileThreads), lds, s, row_ptr, col, perm, ranges,
                       stage_off, counts, stage);
    return hipGetLastError();
}

hipError_t mb_compact_records(const uint32_t* stage_off, const TileMeta* meta, int64_t n_tiles,
                              const unsigned char* stage, unsigned char* rec, hipStream_t s)
{
    if (n_tiles == 0) return hipSuccess;
    hipLaunchKernelGGL(compact_records, dim3((unsigned)n_tiles), dim3(128), 0, s, stage_off, meta, stage, rec);
    return hipGetLastError();
}

hipError_t mb_normal_inverse(bool f64, const int64_t* row_ptr, const int32_t* col, const uint32_t* perm,
                             const void* x, int64_t n, void* out, hipStream_t s)
{
    if (f64)
        hipLaunchKernelGGL(normal_inverse<double>, dim3(blocks_of(n, 256)), dim3(256), 0, s, row_ptr, col, perm,
                           static_cast<const double*>(x), n, 1e-12, static_cast<double*>(out));
    else
        hipLaunchKernelGGL(normal_inverse<float>, dim3(blocks_of(n, 256)), dim3(256), 0, s, row_ptr, col, perm,
                           static_cast<const float*>(x), n, 1e-5, static_cast<float*>(out));
    return hipGetLastError();
}

hipError_t mb_axis_stencil(int dim, bool f64, const void* x, const uint32_t* perm, const int64_t* ring_rp,
                           const int32_t* ring_col, int64_t n, int32_t* slots, uint32_t* cnt, hipStream_t s)
{
    const dim3 g(blocks_of(n, 256)), b(256);
    if (dim == 2) {
        if (f64)
            hipLaunchKernelGGL((axis_slots<2, double>), g, b, 0, s, static_cast<const double*>(x), perm, ring_rp,
                               ring_col, n, slots, cnt);
        else
            hipLaunchKernelGGL((axis_slots<2, float>), g, b, 0, s, static_cast<const float*>(x), perm, ring_rp,
                               ring_col, n, slots, cnt);
    } else {
        if (f64)
            hipLaunchKernelGGL((axis_slots<3, double>), g, b, 0, s, static_cast<const double*>(x), perm, ring_rp,
                               ring_col, n, slots, cnt);
        else
            hipLaunchKernelGGL((axis_slots<3, float>), g, b, 0, s, static_cast<const float*>(x), perm, ring_rp,
                               ring_col, n, slots, cnt);
    }
    return hipGetLastError();
}

hipError_t mb_axis_fill(int dim, const int32_t* slots, const int64_t* row_ptr, int64_t n, int32_t* col, hipStream_t s)
{
    if (dim == 2)
        hipLaunchKernelGGL(axis_fill<2>, dim3(blocks_of(n, 256)), dim3(256), 0, s, slots, row_ptr, n, col);
    else
        hipLaunchKernelGGL(axis_fill<3>, dim3(blocks_of(n, 256)), dim3(256), 0, s, slots, row_ptr, n, col);
    return hipGetLastError();
}

hipError_t mb_transpose_count(const int32_t* col, int64_t nnz, uint32_t* tcnt, hipStream_t s)
{
    if (nnz == 0) return hipSuccess;
    hipLaunchKernelGGL(transpose_count, dim3(blocks_of(nnz, 256)), dim3(256), 0, s, col, nnz, tcnt);
    return hipGetLastError();
}

hipError_t mb_transpose_fill(const int64_t* row_ptr, const int32_t* col, int64_t n, const int64_t* trp, uint32_t* cur,
                             int32_t* tcol, hipStream_t s)
{
    hipLaunchKernelGGL(transpose_fill, dim3(blocks_of(n, 256)), dim3(256), 0, s, row_ptr, col, n, trp, cur, tcol);
    hipLaunchKernelGGL(sort_rows, dim3(blocks_of(n, 256)), dim3(256), 0, s, trp, n, tcol);
    return hipGetLastError();
}

hipError_t mb_csr_compare(const int64_t* rp_a, const int32_t* col_a, const int64_t* rp_b, const int32_t* col_b,
                          int64_t n, int64_t nnz, int* differ, hipStream_t s)
{
    const int64_t m = std::max<int64_t>(n + 1, nnz);
    hipLaunchKernelGGL(csr_compare, dim3(blocks_of(m, 256)), dim3(256), 0, s, rp_a, col_a, rp_b, col_b, n, nnz, differ);
    return hipGetLastError();
}

hipError_t mb_csr_in_count(const int64_t* row_ptr, const int32_t* col, int64_t n, int64_t nnz_in, const uint32_t* perm,
                           uint32_t* cnt, unsigned long long* err, hipStream_t s)
{
    hipLaunchKernelGGL(csr_in_count, dim3(blocks_of(n, 256)), dim3(256), 0, s, row_ptr, col, n, nnz_in, perm, cnt, err);
    return hipGetLastError();
}

hipError_t mb_csr_in_fill(const int64_t* row_ptr, const int32_t* col, int64_t n, const uint32_t* perm,
                          const int32_t* inv, const int64_t* out_rp, int32_t* out, hipStream_t s)
{
    hipLaunchKernelGGL(csr_in_fill, dim3(blocks_of(n, 256)), dim3(256), 0, s, row_ptr, col, n, perm, inv, out_rp, out);
    return hipGetLastError();
}

}  // namespace ftle
