// volume.hip - the steps around the fit that read the CT volume on the device:
// seeding Gaussians from it and ray-marching target images through it
// (Method, "Volumetric Path Tracing" renders the views the peripheral model is
// fitted to; "Periphery Model Training" builds that model from Gaussians
// seeded on the volume's structures).
//
// Seeding: one Gaussian per voxel whose value exceeds the threshold, in raster
// order (vol[ix][iy][iz], flat index (ix n + iy) n + iz); when there are more
// than cap candidates the cap with the smallest priority are kept, still in
// raster order.  Priority of voxel idx: the SplitMix64 output idx + 1 from
// state seed with its low b bits replaced by idx (b = bits of n^3 - 1), so
// priorities are distinct and the kept set is a uniform random subset.  The
// cap-th smallest priority is found on the device (digit histograms, then the few
// candidates that share its first digits), and the kept voxels are written in
// raster order.  Mean = voxel centre, isotropic log-scale, identity rotation, the
// given opacity and the transfer-function colour as degree-0 SH, in double precision
// rounded once to float.  The first hits of rays are capped the same way.
//
// Ray march: one ray per pixel, emission-absorption through the box
// [-1, 1]^3 in float32 - segments of the step length from the box entry (the
// last shortened to the exit), the trilinear sample (zero outside the grid) at
// each segment's midpoint, density t = clamp((v - thr) / range, 0, 1), colour
// lerp(lo, hi, t), alpha = 1 - exp(-extinction t length), stop once T < t_stop;
// RGB = C + T bg, A = 1 - T.
#include <algorithm>
#include <cmath>

#include "gs_internal.h"

namespace gsf {
namespace {

constexpr int kVolBlock = 256;
constexpr int kItemLane = 8;                          // consecutive items of a thread
constexpr int kItemWave = 64 * kItemLane;             // items of a wave
constexpr int kItemTile = 4 * kItemWave;              // items counted and placed together
constexpr int kSelBlock = 1024;                       // threads that histogram and collect
constexpr int kSelList = 512;                         // undecided keys that a workgroup gathers
constexpr int kDigitBits = 10, kDigits = 1 << kDigitBits;
constexpr int kMaxLevels = 6;                         // 60 bits settled: 16 keys at most share them
constexpr int kUndecided = 4096;                      // keys that share the settled digits, at most

__device__ __forceinline__ uint64_t splitmix64(uint64_t state, uint64_t k) {
    uint64_t z = state + k * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t priority(uint64_t seed, uint64_t idx, int ibits) {
    return ((splitmix64(seed, idx + 1ull) >> ibits) << ibits) | idx;
}

// ---- selection of the cap smallest priorities ----------------------------------------
// Items 0 .. n - 1 (voxels, or rays), some of them candidates.  On the device, without
// the host in between:
//   a histogram of the candidates' priorities by their leading 10 bits, and by 10 more
//   within those that it settles, until few enough share them (a further one returns at
//   once where that is so already, as with 2 million candidates of 256^3 voxels);
//   per tile of 2048 items the candidates that are kept for certain, and a list of the
//   undecided;
//   the list resolved, and the tiles' offsets, by one workgroup;
//   the kept items written at their places.
// The list overflows only where priorities crowd: the host sees it after its one
// synchronisation and asks for one digit more.
// The two passes that count read 4 x 16 bytes a lane before they look at any: 20 and 27
// us for 256^3 voxels, of which the 64-bit products of the priorities take about 10 and
// the memory 7 (one load waited for at a time: 24 and 28; workgroups of 256 threads, 8
// a CU, with their 2 million adds to the histogram in memory: 43 and 33; one digit of
// 12 bits: 42 and 27; two of 8 bits: 43 and 21).  Writing: 27 us, resolving 15.
// 500000 voxels of 256^3: 501 us before (eight 8-bit histograms by scalar loads, the
// host waiting for each, and the offsets summed there), 117 now.  20000 first hits of
// 8 x 256 x 256 rays: 473 us before, 278 now.

struct Selection {
    unsigned long long hist[kMaxLevels][kDigits];
    unsigned long long list[kUndecided];
    unsigned long long kstar, kept;   // the largest kept priority; how many are kept
    uint32_t listed, overflow;
};

struct SelArgs {
    int64_t n, cap;
    uint64_t seed;
    int ibits, tiles;
    Selection *sel;
    uint32_t *counts;   // per tile: certainly kept, then the offset of its first kept item
};

// Candidate voxels: those of at least `least`.
struct VoxelItems {
    const uint16_t *vol;
    uint32_t least;
    bool wide;   // 16-byte aligned
    // Bit k: item i + k is a candidate (i a multiple of 8).
    __device__ __forceinline__ uint32_t mask8(int64_t i, int64_t n) const {
        uint32_t m = 0u;
        if (i >= n) return 0u;
        if (wide && i + kItemLane <= n) {
            const uint4 q = *reinterpret_cast<const uint4 *>(vol + i);
            const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
            for (int k = 0; k < 4; k++) {
                m |= (w[k] & 0xFFFFu) >= least ? 1u << (2 * k) : 0u;
                m |= (w[k] >> 16) >= least ? 2u << (2 * k) : 0u;
            }
            return m;
        }
#pragma unroll
        for (int k = 0; k < kItemLane; k++)
            if (i + k < n) m |= (uint32_t)vol[i + k] >= least ? 1u << k : 0u;
        return m;
    }
};

// Candidate rays: those that hit (bytes 0 and 1, room for a multiple of 8 of them).
struct RayItems {
    const uint8_t *hit;
    __device__ __forceinline__ uint32_t mask8(int64_t i, int64_t n) const {
        if (i >= n) return 0u;
        const uint2 q = *reinterpret_cast<const uint2 *>(hit + i);
        uint32_t m = 0u;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            m |= (q.x >> (8 * k) & 1u) << k;
            m |= (q.y >> (8 * k) & 1u) << (4 + k);
        }
        return i + kItemLane <= n ? m : m & ((1u << (int)(n - i)) - 1u);
    }
};

__global__ __launch_bounds__(kVolBlock) void k_select_clear(SelArgs a, int levels) {
    const int i = blockIdx.x * kVolBlock + threadIdx.x;
    if (i < levels * kDigits) (&a.sel->hist[0][0])[i] = 0ull;
    if (i < a.tiles) a.counts[i] = 0u;
    if (i == 0) {
        a.sel->listed = 0u;
        a.sel->overflow = 0u;
    }
}

// Inclusive sum of x over the workgroup's threads up to this one, and the total.
template <int BLOCK, class T>
__device__ __forceinline__ T block_scan(T x, T &total) {
    __shared__ T s_sum[BLOCK / 64];
    const int lane = (int)threadIdx.x & 63, w = (int)threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const T y = __shfl_up(x, o, 64);
        if (lane >= o) x += y;
    }
    __syncthreads();   // the sums of an earlier scan have been read
    if (lane == 63) s_sum[w] = x;
    __syncthreads();
    total = 0;
#pragma unroll
    for (int k = 0; k < BLOCK / 64; k++) {
        if (k < w) x += s_sum[k];
        total += s_sum[k];
    }
    return x;
}

struct Pick {
    uint64_t prefix;   // the settled digits of the cap-th smallest priority
    int64_t rank;      // its 1-based rank among the candidates that share them
    int levels;        // how many digits are settled
    bool all;          // every candidate is kept
    bool few;          // or those that share the digits fit the list
};

// The digit in which the histogram's running sum reaches rank, which drops by the sum
// before it; its count, and the histogram's total.  Called by every thread of the
// workgroup.
template <int BLOCK, class T>
__device__ __forceinline__ int find_digit(const T *hist, int64_t &rank, int64_t &count, int64_t &total) {
    constexpr int kPer = kDigits / BLOCK;
    __shared__ int s_digit;
    __shared__ int64_t s_rank, s_count;
    unsigned long long own = 0ull, sum;
#pragma unroll
    for (int k = 0; k < kPer; k++) own += hist[threadIdx.x * kPer + k];
    int64_t before = (int64_t)(block_scan<BLOCK>(own, sum) - own);
    total = (int64_t)sum;
    const int64_t want = rank < total ? rank : total;
    if (before < want && before + (int64_t)own >= want) {
        int k = 0;
        int64_t h;
        for (; before + (h = (int64_t)hist[threadIdx.x * kPer + k]) < want; k++) before += h;
        s_digit = (int)threadIdx.x * kPer + k;
        s_rank = rank - before;
        s_count = h;
    }
    __syncthreads();
    const int d = total ? s_digit : 0;
    count = total ? s_count : 0;
    if (total) rank = s_rank;
    __syncthreads();
    return d;
}

__device__ __forceinline__ int digit_shift(int level) { return 64 - kDigitBits * (level + 1); }

template <int BLOCK>
__device__ __forceinline__ Pick pick(const SelArgs &a, int levels) {
    Pick p{0ull, a.cap, 0, false, false};
    while (p.levels < levels && !p.all && !p.few) {
        int64_t count, total;
        const int d = find_digit<BLOCK>(a.sel->hist[p.levels], p.rank, count, total);
        p.all = p.levels == 0 && total <= a.cap;
        p.few = count <= kUndecided;
        p.prefix |= (uint64_t)d << digit_shift(p.levels++);
    }
    return p;
}

// Calls f(k, priority) for each of the thread's candidates first + k.
template <class F>
__device__ __forceinline__ void for_keys(uint32_t mask, int64_t first, const SelArgs &a, F f) {
#pragma unroll
    for (int k = 0; k < kItemLane; k++)
        if (mask >> k & 1u) f(k, priority(a.seed, (uint64_t)(first + k), a.ibits));
}

// Calls f(tile, first item, candidates) for each wave's 512 items, four of them read
// at a time, far apart as candidates cluster.
template <class ITEMS, class F>
__device__ __forceinline__ void for_waves(const ITEMS &items, const SelArgs &a, F f) {
    const int64_t waves = 4 * (int64_t)a.tiles, stride = (int64_t)gridDim.x * (kSelBlock / 64);
    for (int64_t c = (int64_t)blockIdx.x * (kSelBlock / 64) + (threadIdx.x >> 6); c < waves; c += 4 * stride) {
        const int64_t lane0 = (threadIdx.x & 63) * kItemLane;
        uint32_t m[4];
#pragma unroll
        for (int q = 0; q < 4; q++) m[q] = items.mask8((c + q * stride) * kItemWave + lane0, a.n);
#pragma unroll 1
        for (int q = 0; q < 4; q++) {
            const uint32_t mq = q == 0 ? m[0] : (q == 1 ? m[1] : (q == 2 ? m[2] : m[3]));
            if (__builtin_amdgcn_ballot_w64(mq != 0u) == 0ull) continue;
            f((int)((c + q * stride) >> 2), (c + q * stride) * kItemWave + lane0, mq);
        }
    }
}

// Histogram of the digit after `level` settled ones.
template <class ITEMS>
__global__ __launch_bounds__(kSelBlock) void k_select_hist(ITEMS items, SelArgs a, int level) {
    __shared__ uint32_t h[kDigits];
    Pick p{};
    if (level) {
        p = pick<kSelBlock>(a, level);
        if (p.all || p.few) return;
    }
    for (int d = threadIdx.x; d < kDigits; d += kSelBlock) h[d] = 0u;
    __syncthreads();
    const int shift = digit_shift(level);
    for_waves(items, a, [&](int, int64_t first, uint32_t m) {
        for_keys(m, first, a, [&](int, uint64_t key) {
            if (level == 0 || ((key ^ p.prefix) >> (shift + kDigitBits)) == 0ull)
                atomicAdd(&h[(key >> shift) & (kDigits - 1)], 1u);
        });
    });
    __syncthreads();
    for (int d = threadIdx.x; d < kDigits; d += kSelBlock)
        if (h[d]) atomicAdd(&a.sel->hist[level][d], (unsigned long long)h[d]);
}

// Per tile the candidates that are kept for certain: those whose settled digits are
// below the cap-th's, or all of them.  Those that share its digits go to the list.
template <class ITEMS>
__global__ __launch_bounds__(kSelBlock) void k_select_collect(ITEMS items, SelArgs a, int levels) {
    __shared__ unsigned long long s_key[kSelList];
    __shared__ uint32_t s_listed, s_at;
    if (threadIdx.x == 0) s_listed = 0u;
    const Pick p = pick<kSelBlock>(a, levels);
    __syncthreads();
    const int shift = digit_shift(p.levels - 1);
    const uint64_t want = p.prefix >> shift;
    for_waves(items, a, [&](int t, int64_t first, uint32_t m) {
        uint32_t c = 0u;
        if (p.all) c = __popc(m);
        else
            for_keys(m, first, a, [&](int, uint64_t key) {
                const uint64_t top = key >> shift;
                c += top < want ? 1u : 0u;
                if (top != want) return;
                uint32_t at = atomicAdd(&s_listed, 1u);
                if (at < kSelList) {
                    s_key[at] = key;
                    return;
                }
                at = atomicAdd(&a.sel->listed, 1u);
                if (at < kUndecided) a.sel->list[at] = key;
            });
#pragma unroll
        for (int o = 32; o; o >>= 1) c += __shfl_xor(c, o, 64);
        if ((threadIdx.x & 63) == 0 && c) atomicAdd(&a.counts[t], c);
    });
    __syncthreads();
    const uint32_t n = min(s_listed, (uint32_t)kSelList);
    if (threadIdx.x == 0 && n) s_at = atomicAdd(&a.sel->listed, n);
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < n; i += kSelBlock)
        if (s_at + i < kUndecided) a.sel->list[s_at + i] = s_key[i];
}

// One workgroup: the largest kept priority from the list, its kept keys counted in
// their tiles, and the tiles' counts turned into offsets.  host: {kept, overflow}.
__global__ __launch_bounds__(1024) void k_select_finish(SelArgs a, int levels, unsigned long long *host) {
    __shared__ unsigned long long s_key[kUndecided];
    constexpr int kTiles = 4096;
    __shared__ uint32_t s_hist[kTiles];   // a digit's; then of 4096 tiles at a time, the list's kept keys
    const int t = (int)threadIdx.x;
    const Pick p = pick<1024>(a, levels);
    const uint32_t listed = p.all ? 0u : a.sel->listed;
    if (listed > kUndecided) {
        if (t == 0) {
            a.sel->overflow = 1u;
            host[0] = 0ull;
            host[1] = 1ull;
        }
        return;
    }
    uint64_t kstar = ~0ull;
    if (!p.all) {
        for (uint32_t i = t; i < listed; i += 1024) s_key[i] = a.sel->list[i];
        uint64_t prefix = p.prefix, settled = ~0ull << digit_shift(p.levels - 1);
        int64_t rank = p.rank;
        for (int level = p.levels; ~settled; level++) {
            const int shift = max(digit_shift(level), 0);   // (the last digit takes settled bits along)
            for (int d = t; d < kDigits; d += 1024) s_hist[d] = 0u;
            __syncthreads();
            for (uint32_t i = t; i < listed; i += 1024)
                if (((s_key[i] ^ prefix) & settled) == 0ull)
                    atomicAdd(&s_hist[(s_key[i] >> shift) & (kDigits - 1)], 1u);
            __syncthreads();
            int64_t count, total;
            const int d = find_digit<1024>(s_hist, rank, count, total);
            prefix |= (uint64_t)d << shift;
            settled |= (uint64_t)(kDigits - 1) << shift;
            if (count == rank) break;   // all that share the digits are kept
        }
        kstar = prefix | ~settled;
    }
    const uint64_t imask = (1ull << a.ibits) - 1ull;
    uint32_t sum = 0u;
    for (int base = 0; base < a.tiles; base += kTiles) {
        for (int k = t; k < kTiles; k += 1024) s_hist[k] = 0u;
        __syncthreads();
        for (uint32_t i = t; i < listed; i += 1024) {
            const int64_t tile = (int64_t)((s_key[i] & imask) / kItemTile) - base;
            if (s_key[i] <= kstar && tile >= 0 && tile < kTiles) atomicAdd(&s_hist[tile], 1u);
        }
        __syncthreads();
        const int first = base + t * 4;
        uint32_t c[4], own = 0u, total;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            c[k] = first + k < a.tiles ? a.counts[first + k] + s_hist[t * 4 + k] : 0u;
            own += c[k];
        }
        uint32_t at = sum + block_scan<1024>(own, total) - own;
        sum += total;
#pragma unroll
        for (int k = 0; k < 4; k++)
            if (first + k < a.tiles) {
                a.counts[first + k] = at;
                at += c[k];
            }
    }
    if (t == 0) {
        a.sel->kstar = kstar;
        a.sel->kept = sum;
        host[0] = sum;
        host[1] = 0ull;
    }
}

// The kept items in order: put(item of the tile, its place, the number of them all).
template <class ITEMS, class PUT>
__global__ __launch_bounds__(kVolBlock) void k_select_emit(ITEMS items, SelArgs a, PUT put) {
    __shared__ uint16_t s_item[kItemTile];
    if (a.sel->overflow) return;
    const int t = blockIdx.x;
    const int64_t m = (int64_t)a.sel->kept, at = a.counts[t];
    if (at == (t + 1 < a.tiles ? (int64_t)a.counts[t + 1] : m)) return;
    const uint64_t kstar = a.sel->kstar;
    const int64_t base = (int64_t)t * kItemTile, first = base + threadIdx.x * kItemLane;
    uint32_t keep = 0u, total;
    for_keys(items.mask8(first, a.n), first, a, [&](int k, uint64_t key) { keep |= key <= kstar ? 1u << k : 0u; });
    uint32_t r = block_scan<kVolBlock>((uint32_t)__popc(keep), total) - __popc(keep);
#pragma unroll
    for (int k = 0; k < kItemLane; k++)
        if (keep >> k & 1u) s_item[r++] = (uint16_t)(threadIdx.x * kItemLane + k);
    __syncthreads();
    const PUT put_t = put.at_tile(base);
    for (uint32_t i = threadIdx.x; i < total; i += kVolBlock) put_t((int)s_item[i], at + i, m);
}

// A kept voxel's Gaussian, planar [14][m].
struct PutVoxel {
    const uint16_t *vol;
    float *P;
    double inv_n2;          // 2 / n
    double thr, range;
    double lo[3], hi[3];
    double sh_dc;           // value of the constant SH basis function
    float log_scale, logit_opacity, inv_n;
    int n;
    int64_t base;           // the tile's first voxel, (x0, y0, z0)
    int x0, y0, z0;

    __device__ __forceinline__ PutVoxel at_tile(int64_t first) const {
        PutVoxel p = *this;
        p.base = first;
        const int64_t row = first / n;
        p.z0 = (int)(first - row * n);
        p.x0 = (int)(row / n);
        p.y0 = (int)(row - (int64_t)p.x0 * n);
        return p;
    }
    // j / n for 0 <= j < n + kItemTile: half a unit is far more than the rounding.
    __device__ __forceinline__ int over_n(int j) const { return (int)(((float)j + 0.5f) * inv_n); }
    __device__ __forceinline__ void operator()(int item, int64_t at, int64_t m) const {
        const int row = over_n(z0 + item), iz = z0 + item - row * n;
        const int plane = over_n(y0 + row), iy = y0 + row - plane * n, ix = x0 + plane;
        const double t0 = ((double)vol[base + item] - thr) / range;
        const double t = t0 < 0.0 ? 0.0 : (t0 > 1.0 ? 1.0 : t0);
        float *p = P + at;
        p[0 * m] = (float)(((double)ix + 0.5) * inv_n2 - 1.0);
        p[1 * m] = (float)(((double)iy + 0.5) * inv_n2 - 1.0);
        p[2 * m] = (float)(((double)iz + 0.5) * inv_n2 - 1.0);
        p[3 * m] = p[4 * m] = p[5 * m] = log_scale;
        p[6 * m] = 1.f;
        p[7 * m] = p[8 * m] = p[9 * m] = 0.f;
        p[10 * m] = logit_opacity;
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            const double col = lo[ch] * (1.0 - t) + hi[ch] * t;
            p[(11 + ch) * m] = (float)((col - 0.5) / sh_dc);
        }
    }
};

// A kept ray's Gaussian, planar [14][m], and its number (ray_ids nullable).
struct PutHit {
    const float4 *pos, *col;
    float *P;
    int32_t *ray_ids;
    float log_scale, logit_opacity, inv_sh_dc;
    int64_t base;

    __device__ __forceinline__ PutHit at_tile(int64_t first) const {
        PutHit p = *this;
        p.base = first;
        return p;
    }
    __device__ __forceinline__ void operator()(int item, int64_t at, int64_t m) const {
        const int64_t i = base + item;
        const float4 p4 = pos[i], c4 = col[i];
        float *p = P + at;
        p[0 * m] = p4.x;
        p[1 * m] = p4.y;
        p[2 * m] = p4.z;
        p[3 * m] = p[4 * m] = p[5 * m] = log_scale;
        p[6 * m] = 1.f;
        p[7 * m] = p[8 * m] = p[9 * m] = 0.f;
        p[10 * m] = logit_opacity;
        p[11 * m] = (c4.x - 0.5f) * inv_sh_dc;
        p[12 * m] = (c4.y - 0.5f) * inv_sh_dc;
        p[13 * m] = (c4.z - 0.5f) * inv_sh_dc;
        if (ray_ids) ray_ids[at] = (int32_t)i;
    }
};

// ---- ray march ---------------------------------------------------------------------
// Both marches sample the volume about twice a voxel along every pixel's ray.  Most
// of that space is empty (below the transfer function's threshold), and a ray is a
// serial chain of gathers, so one thread per ray that takes each segment in turn
// spends its time on reads that change nothing, and ends with the longest rays alone
// on the chip.  Here
// - a grid of at most 128^3 cells, made from the volume first in every call (one pass
//   over it), says which cells hold a voxel that can matter; a 64-bit word is a 4 x 4
//   x 4 block of cells, so that one read gives both levels to skip by.  (64^3 cells:
//   raymarch 3% slower, first hits the same.)  It is read through the cache: held in
//   LDS it took workgroups of several waves, which wait for their longest ray (2550
//   us with 8 waves, 1680 with 4, 1390 with one and no LDS);
// - a wave holds an 8 x 8 square of pixels, and its lanes fall out of step: some look
//   for the next occupied cell, others have segments to read.  In every turn it does
//   what more of them wait for.  (All look, then all read: 1330 us.)
// - four segments are read at a time, so that their loads are in flight together (two:
//   890 us, first hits 184), the two corners along z with one load.  (Four lanes
//   to a ray, a segment each: 2320 us, as they look for it four times over.)
// What is skipped has density zero exactly and every sum keeps its order: the images
// are the same bits.  4 views of 1024 x 1024 through 256^3: 4 x 3856 us before, 816 now;
// first hits of 8 x 256 x 256 rays through 128^3: 731 us before, 145 now.  What is left
// is issue of vector instructions in the lanes that still differ (about 60% work).

constexpr int kOccSide = 128;   // cells per side at most

struct OccGrid {
    const uint2 *occ;       // [blocks][blocks][blocks], 4 x 4 x 4 cells each; null: every cell is occupied
    float size, inv_size;   // voxels per cell side
    int last, blocks;       // cells per side - 1; blocks of cells per side
};

// Cells of side `size` voxels: cell c holds the samples whose lower corner i has
// i + 1 in [c size, (c + 1) size), so its corners are the voxels c size - 1 ..
// (c + 1) size - 1.  A cell is occupied when one of them is above zero and reaches
// `least` (the threshold, less what rounding may add to an interpolated value).
// Bit 16 (cx & 3) + 4 (cy & 3) + (cz & 3) of its block's 64.  One workgroup per plane
// cx of a column of blocks, one wave per row of cells (cx, cy): its lanes take pairs
// of voxels along z and their maximum over the row's lines.
__global__ __launch_bounds__(256) void k_occupancy(const uint16_t *__restrict__ vol, int n, int size, int cells,
                                                   float least, uint16_t *__restrict__ occ) {
    __shared__ uint16_t zmax[4][2048 + 2];
    __shared__ uint64_t bits[4][(kOccSide + 63) / 64];
    const int blocks = (cells + 3) >> 2, cx = blockIdx.x / blocks, by = blockIdx.x - cx * blocks;
    const int w = (int)threadIdx.x >> 6, lane = (int)threadIdx.x & 63, cy = 4 * by + w;
    const int x0 = max(cx * size - 1, 0), x1 = min(cx * size + size - 1, n - 1);   // none past the last cell
    const int y0 = max(cy * size - 1, 0), y1 = min(cy * size + size - 1, n - 1);
    for (int z = 2 * lane; z < n; z += 128) {
        const bool pair = z + 1 < n;
        uint32_t m0 = 0u, m1 = 0u;
        for (int x = x0; x <= x1; x++)
            for (int y = y0; y <= y1; y++) {
                const uint16_t *p = vol + ((int64_t)x * n + y) * n + z;
                uint32_t q = 0u;
                if (pair) __builtin_memcpy(&q, p, 4);
                else q = *p;
                m0 = max(m0, q & 0xFFFFu);
                m1 = max(m1, q >> 16);
            }
        zmax[w][z] = (uint16_t)m0;
        if (pair) zmax[w][z + 1] = (uint16_t)m1;
    }
    __syncthreads();
    for (int c0 = 0; c0 < cells; c0 += 64) {
        const int cz = c0 + lane, z1 = min(cz * size + size - 1, n - 1);
        uint32_t m = 0u;
        for (int z = max(cz * size - 1, 0); z <= z1; z++) m = max(m, (uint32_t)zmax[w][z]);
        const uint64_t full = __builtin_amdgcn_ballot_w64(m > 0u && (float)m >= least);
        if (lane == 0) bits[w][c0 >> 6] = full;
    }
    __syncthreads();
    if ((int)threadIdx.x >= blocks) return;
    const int bz = (int)threadIdx.x;
    uint32_t h = 0u;
#pragma unroll
    for (int r = 0; r < 4; r++) h |= ((uint32_t)(bits[r][bz >> 4] >> (4 * (bz & 15))) & 15u) << (4 * r);
    occ[4 * (((int64_t)(cx >> 2) * blocks + by) * blocks + bz) + (cx & 3)] = (uint16_t)h;
}

struct MarchConst {
    int n, color_steps;
    float step, extinction, t_stop, thr, inv_range, hit_alpha;
    float lo[3], hi[3];
};

constexpr int kMarchU = 4;   // segments read at a time
constexpr int kMarchX = 8, kMarchY = 8, kMarchBlock = kMarchX * kMarchY;   // pixels of a workgroup

struct RayViews {
    int64_t off[kMaxViews + 1];   // first ray of each view (rays in view, row, column order)
    int32_t block[kMaxViews + 1]; // its first workgroup
    int32_t width[kMaxViews], height[kMaxViews];
    int nviews;
};

__device__ __forceinline__ float vol_at(const uint16_t *__restrict__ vol, int n, int i, int j, int k) {
    return (i < 0 || i >= n || j < 0 || j >= n || k < 0 || k >= n) ? 0.f
                                                                       : (float)vol[((int64_t)i * n + j) * n + k];
}

// One ray of a march: pixel (i, j)'s, its interval in the box and the steps it
// takes through it.
struct Ray {
    float o[3], d[3], t0, t1;
    float inv_du[3];   // steps per voxel along each axis
    bool meets;        // the box
};

__device__ __forceinline__ Ray make_ray(const gsf_camera *__restrict__ cam, int i, int j, const MarchConst &mc) {
    Ray r;
    const float *Rm = cam->viewmat;   // rows of [R | t]
    const float dc0 = ((float)i + 0.5f - cam->cx) / cam->fx, dc1 = ((float)j + 0.5f - cam->cy) / cam->fy;
#pragma unroll
    for (int a = 0; a < 3; a++) r.d[a] = Rm[a] * dc0 + Rm[4 + a] * dc1 + Rm[8 + a];
    const float inn = 1.f / sqrtf(r.d[0] * r.d[0] + r.d[1] * r.d[1] + r.d[2] * r.d[2]);
    r.t0 = -INFINITY;
    r.t1 = INFINITY;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        r.o[a] = cam->campos[a];
        r.d[a] *= inn;
        const float inv = 1.f / r.d[a];
        float ta = (-1.f - r.o[a]) * inv, tb = (1.f - r.o[a]) * inv;
        if (ta > tb) { const float tmp = ta; ta = tb; tb = tmp; }
        r.t0 = fmaxf(r.t0, ta);
        r.t1 = fminf(r.t1, tb);
        r.inv_du[a] = 1.f / (r.d[a] * (0.5f * (float)mc.n) * mc.step);
    }
    r.t0 = fmaxf(r.t0, 0.f);
    r.meets = r.t1 > r.t0;
    return r;
}

// Segment k of the ray: its length and the voxel coordinates of its midpoint
// (mid: the distance there); false past the exit.
__device__ __forceinline__ bool segment(const Ray &r, const MarchConst &mc, int k, float &len, float &mid,
                                        float (&u)[3]) {
    const float s0 = r.t0 + (float)k * mc.step;
    const float s1 = fminf(s0 + mc.step, r.t1);
    if (!(s1 > s0)) return false;
    len = s1 - s0;
    mid = 0.5f * (s0 + s1);
    const float h = 0.5f * (float)mc.n;
#pragma unroll
    for (int a = 0; a < 3; a++) u[a] = (r.o[a] + r.d[a] * mid + 1.f) * h - 0.5f;
    return true;
}

// Looks segment k's midpoint up in the grid.  In an occupied cell, end: the segments
// up to there are read before the grid is looked at again.  In an empty cell, or an
// empty block of them, k moves past the segments that lie in it too: the whole steps
// left to the nearest of its faces, kept 1/100 voxel short of it, far more than the
// rounding of a sample's coordinates.  False past the exit.
__device__ __forceinline__ bool look(const Ray &r, const MarchConst &mc, const OccGrid &og, int &k, int &end) {
    float len, mid, u[3];
    if (!segment(r, mc, k, len, mid, u)) return false;
    if (!og.occ) {
        end = 0x7FFFFF00;
        return true;
    }
    // (the half keeps the quotient away from whole numbers; samples a rounding
    // outside the volume belong to the nearest cell)
    int c[3];
#pragma unroll
    for (int a = 0; a < 3; a++) c[a] = min(max((int)((floorf(u[a]) + 1.5f) * og.inv_size), 0), og.last);
    const uint2 word = og.occ[((c[0] >> 2) * og.blocks + (c[1] >> 2)) * og.blocks + (c[2] >> 2)];
    const bool block = (word.x | word.y) == 0u;
    const float size = block ? 4.f * og.size : og.size;
    float left = 1e6f;
#pragma unroll
    for (int a = 0; a < 3; a++) {
        const float face = (float)(block ? c[a] >> 2 : c[a]) * size + (r.inv_du[a] > 0.f ? size - 1.01f : -0.99f);
        left = fminf(left, (face - u[a]) * r.inv_du[a]);
    }
    const int next = k + max((int)left, 0) + 1;
    const uint32_t half = (c[0] & 2) ? word.y : word.x;
    if ((half >> (((c[0] & 1) << 4) + ((c[1] & 3) << 2) + (c[2] & 3))) & 1u) end = next;
    else k = next;
    return true;
}

// Whether the wave reads segments next (the lanes that have some: k < end), or looks
// at the grid (the others): what more of its rays wait for.  In turns of one and then
// the other, each until the last ray was through, a third to a half of the lanes worked.
__device__ __forceinline__ bool reads_next(bool go, int k, int end) {
    return 2 * __popcll(__builtin_amdgcn_ballot_w64(go && k < end)) > __popcll(__builtin_amdgcn_ballot_w64(go));
}

__device__ __forceinline__ float lerp8(const float (&v)[8], float fx, float fy, float fz) {
    const float c00 = v[0] * (1.f - fz) + v[1] * fz, c01 = v[2] * (1.f - fz) + v[3] * fz;
    const float c10 = v[4] * (1.f - fz) + v[5] * fz, c11 = v[6] * (1.f - fz) + v[7] * fz;
    const float c0 = c00 * (1.f - fy) + c01 * fy, c1 = c10 * (1.f - fy) + c11 * fy;
    return c0 * (1.f - fx) + c1 * fx;
}

// Densities t of segments k .. k + kMarchU - 1 at their midpoints (trilinear, zero
// outside the volume), with their lengths and distances; ok[e] false past the exit.
// The loads of all of them are in flight together: inside the volume two corners
// along z are read as one 32-bit word; where some lane's sample has a corner
// outside, every corner by itself.
__device__ __forceinline__ void sample_run(const uint16_t *__restrict__ vol, const Ray &r, const MarchConst &mc,
                                           int k, bool (&ok)[kMarchU], float (&len)[kMarchU],
                                           float (&mid)[kMarchU], float (&t)[kMarchU]) {
    const int n = mc.n;
    float f[kMarchU][3];
    int i0[kMarchU][3];
    bool inner = true;
#pragma unroll
    for (int e = 0; e < kMarchU; e++) {
        float u[3] = {0.f, 0.f, 0.f};
        len[e] = mid[e] = 0.f;
        ok[e] = segment(r, mc, k + e, len[e], mid[e], u);
#pragma unroll
        for (int a = 0; a < 3; a++) {
            const float f0 = floorf(u[a]);
            f[e][a] = u[a] - f0;
            i0[e][a] = (int)f0;
            inner &= !ok[e] || (i0[e][a] >= 0 && i0[e][a] < n - 1);
        }
    }
    float val[kMarchU];
    if (__builtin_amdgcn_ballot_w64(!inner) == 0ull) {
        uint32_t q[kMarchU][4];
        const int64_t plane = (int64_t)n * n;
#pragma unroll
        for (int e = 0; e < kMarchU; e++) {
            if (!ok[e]) continue;
            const uint16_t *p = vol + ((int64_t)(i0[e][0] * n + i0[e][1]) * n + i0[e][2]);
            __builtin_memcpy(&q[e][0], p, 4);
            __builtin_memcpy(&q[e][1], p + n, 4);
            __builtin_memcpy(&q[e][2], p + plane, 4);
            __builtin_memcpy(&q[e][3], p + plane + n, 4);
        }
#pragma unroll
        for (int e = 0; e < kMarchU; e++) {
            float v[8];
#pragma unroll
            for (int w = 0; w < 4; w++) {
                v[2 * w] = (float)(q[e][w] & 0xFFFFu);
                v[2 * w + 1] = (float)(q[e][w] >> 16);
            }
            val[e] = lerp8(v, f[e][0], f[e][1], f[e][2]);
        }
    } else {
#pragma unroll 1
        for (int e = 0; e < kMarchU; e++) {
            float v[8];
#pragma unroll
            for (int w = 0; w < 8; w++)
                v[w] = ok[e] ? vol_at(vol, n, i0[e][0] + (w >> 2), i0[e][1] + ((w >> 1) & 1), i0[e][2] + (w & 1)) : 0.f;
            val[e] = lerp8(v, f[e][0], f[e][1], f[e][2]);
        }
    }
#pragma unroll
    for (int e = 0; e < kMarchU; e++) t[e] = fminf(fmaxf((val[e] - mc.thr) * mc.inv_range, 0.f), 1.f);
}

// The thread's view and pixel (false: outside the view), and the grid into LDS.
__device__ __forceinline__ bool march_pixel(const RayViews &rv, int &v, int &i, int &j) {
    v = 0;
    while (v + 1 < rv.nviews && (int)blockIdx.x >= rv.block[v + 1]) v++;
    const int b = (int)blockIdx.x - rv.block[v], bx = (rv.width[v] + kMarchX - 1) / kMarchX;
    const int lane = (int)threadIdx.x;
    i = (b % bx) * kMarchX + (lane & 7);
    j = (b / bx) * kMarchY + (lane >> 3);
    return i < rv.width[v] && j < rv.height[v];
}

__global__ __launch_bounds__(kMarchBlock) void k_raymarch(const uint16_t *__restrict__ vol,
                                                          const gsf_camera *__restrict__ cams, RayViews rv,
                                                          MarchConst mc, OccGrid og, float *__restrict__ out) {
    int v, i, j;
    if (!march_pixel(rv, v, i, j)) return;
    const gsf_camera *cam = cams + v;
    const Ray r = make_ray(cam, i, j, mc);
    float C[3] = {0.f, 0.f, 0.f}, T = 1.f;
    bool go = r.meets;
    int k = 0, end = 0;
    while (go) {
        if (!reads_next(go, k, end)) {
            if (k >= end) go = look(r, mc, og, k, end);
            continue;
        }
        if (k >= end) continue;
        bool ok[kMarchU];
        float len[kMarchU], mid[kMarchU], t[kMarchU];
        sample_run(vol, r, mc, k, ok, len, mid, t);
#pragma unroll
        for (int e = 0; e < kMarchU; e++) {
            if (!(go && ok[e] && t[e] > 0.f)) continue;
            const float alpha = 1.f - expf(-mc.extinction * t[e] * len[e]);
#pragma unroll
            for (int c = 0; c < 3; c++) C[c] += (mc.lo[c] * (1.f - t[e]) + mc.hi[c] * t[e]) * alpha * T;
            T *= 1.f - alpha;
            go = !(T < mc.t_stop);
        }
        go &= ok[kMarchU - 1];
        k += kMarchU;
    }
    const int64_t plane = (int64_t)rv.width[v] * rv.height[v], q = (int64_t)j * rv.width[v] + i;
    float *o = out + 4 * rv.off[v];
#pragma unroll
    for (int c = 0; c < 3; c++) o[c * plane + q] = C[c] + T * cam->bg[c];
    o[3 * plane + q] = 1.f - T;
}

// ---- first-hit point cloud ----------------------------------------------------------
// The paper seeds its initial cloud from the first significant hit of rays
// cast at the volume from viewpoints around it, each point coloured by the
// path tracer (Method, "Volumetric Path Tracing").  Here a ray's hit is the
// midpoint of the first march segment after which the accumulated opacity
// reaches hit_alpha, and its colour the emission-absorption colour of that
// segment and the next color_steps - 1, divided by their opacity.

__global__ __launch_bounds__(kMarchBlock) void k_first_hit(const uint16_t *__restrict__ vol,
                                                           const gsf_camera *__restrict__ cams, RayViews rv,
                                                           MarchConst mc, OccGrid og, uint8_t *__restrict__ hit,
                                                           float4 *__restrict__ pos, float4 *__restrict__ col) {
    int v, i, j;
    if (!march_pixel(rv, v, i, j)) return;
    const int64_t ray = rv.off[v] + (int64_t)j * rv.width[v] + i;
    const Ray r = make_ray(cams + v, i, j, mc);
    hit[ray] = 0;
    if (!r.meets) return;
    float T = 1.f, mid_hit = 0.f;
    int khit = -1;
    bool go = true;
    int k = 0, end = 0;
    while (go) {
        if (!reads_next(go, k, end)) {
            if (k >= end) go = look(r, mc, og, k, end);
            continue;
        }
        if (k >= end) continue;
        bool ok[kMarchU];
        float len[kMarchU], mid[kMarchU], t[kMarchU];
        sample_run(vol, r, mc, k, ok, len, mid, t);
#pragma unroll
        for (int e = 0; e < kMarchU; e++) {
            if (!(go && ok[e])) continue;
            T *= expf(-mc.extinction * t[e] * len[e]);
            if (1.f - T >= mc.hit_alpha) {
                khit = k + e;
                mid_hit = mid[e];
                go = false;
            }
        }
        go &= ok[kMarchU - 1];
        k += kMarchU;
    }
    if (khit < 0) return;
    float C[3] = {0.f, 0.f, 0.f}, Ts = 1.f;
    for (k = khit; k < khit + mc.color_steps; k += kMarchU) {
        bool ok[kMarchU];
        float len[kMarchU], mid[kMarchU], t[kMarchU];
        sample_run(vol, r, mc, k, ok, len, mid, t);
#pragma unroll
        for (int e = 0; e < kMarchU; e++) {
            if (!(ok[e] && k + e < khit + mc.color_steps)) continue;
            const float alpha = 1.f - expf(-mc.extinction * t[e] * len[e]);
#pragma unroll
            for (int c = 0; c < 3; c++) C[c] += (mc.lo[c] * (1.f - t[e]) + mc.hi[c] * t[e]) * alpha * Ts;
            Ts *= 1.f - alpha;
        }
        if (!ok[kMarchU - 1]) break;
    }
    const float ia = 1.f / (1.f - Ts);
    hit[ray] = 1;
    pos[ray] = make_float4(r.o[0] + r.d[0] * mid_hit, r.o[1] + r.d[1] * mid_hit, r.o[2] + r.d[2] * mid_hit, 0.f);
    col[ray] = make_float4(C[0] * ia, C[1] * ia, C[2] * ia, 0.f);
}

}  // namespace

namespace {
size_t occupancy_bytes() { return (size_t)kOccSide * kOccSide * kOccSide / 8; }

int item_tiles(int64_t n) { return (int)((n + kItemTile - 1) / kItemTile); }

// The items of the cap smallest priorities, written by `put`; their number to *count.
// counts: item_tiles(n); synchronises the stream.
template <class ITEMS, class PUT>
hipError_t run_select(hipStream_t s, const ITEMS &items, const PUT &put, int64_t n, int64_t cap, uint64_t seed,
                      uint32_t *counts, const VolumeScratch &vs, int cus, int64_t *count) {
    SelArgs a{};
    a.n = n;
    a.cap = cap;
    a.seed = seed;
    while ((int64_t(1) << a.ibits) < n) a.ibits++;
    if (a.ibits < 1) a.ibits = 1;
    a.tiles = item_tiles(n);
    a.sel = (Selection *)((char *)vs.device + occupancy_bytes());
    a.counts = counts;
    const int grid = std::min((4 * a.tiles + kSelBlock / 64 - 1) / (kSelBlock / 64), 2 * cus);   // what the device holds
    int levels = 1;
    while (levels < kMaxLevels && (n >> (kDigitBits * levels)) > kUndecided) levels++;
    for (;; levels++) {
        k_select_clear<<<(std::max(levels * kDigits, a.tiles) + kVolBlock - 1) / kVolBlock, kVolBlock, 0, s>>>(a, levels);
        for (int l = 0; l < levels; l++) k_select_hist<<<grid, kSelBlock, 0, s>>>(items, a, l);
        k_select_collect<<<grid, kSelBlock, 0, s>>>(items, a, levels);
        k_select_finish<<<1, 1024, 0, s>>>(a, levels, vs.host);
        k_select_emit<<<a.tiles, kVolBlock, 0, s>>>(items, a, put);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (!vs.host[1] || levels == kMaxLevels) break;
    }
    *count = (int64_t)vs.host[0];
    return hipSuccess;
}
}  // namespace

// Host side of the seeding (synchronises the stream).
hipError_t run_seed(hipStream_t s, const uint16_t *vol, int n, double thr, double range,
                    const double *lo, const double *hi, double opacity, int64_t cap, uint64_t seed,
                    float *params, int64_t *count, void *scratch, const VolumeScratch &vs, int cus) {
    if (!vs.device) return hipErrorStreamCaptureUnsupported;   // the call synchronises
    const int64_t nvox = (int64_t)n * n * n;
    VoxelItems items{};
    items.vol = vol;
    const float thr_f = (float)thr;   // value > thr_f, for whole values
    items.least = thr_f < 0.f ? 0u : (thr_f < 65535.f ? (uint32_t)thr_f + 1u : 65536u);   // NaN: none
    items.wide = ((uintptr_t)vol & 15u) == 0;
    PutVoxel put{};
    put.vol = vol;
    put.P = params;
    put.n = n;
    put.inv_n = 1.f / (float)n;
    put.inv_n2 = 2.0 / n;
    put.thr = thr;
    put.range = range;
    for (int c = 0; c < 3; c++) {
        put.lo[c] = lo[c];
        put.hi[c] = hi[c];
    }
    put.sh_dc = 0.5 / std::sqrt(std::acos(-1.0));
    put.log_scale = (float)std::log(2.0 / n);
    put.logit_opacity = (float)std::log(opacity / (1.0 - opacity));
    uint32_t *counts = (uint32_t *)((char *)scratch + 256 * sizeof(unsigned long long));
    return run_select(s, items, put, nvox, cap, seed, counts, vs, cus, count);
}

size_t seed_scratch_bytes(int64_t nvox) { return 256 * sizeof(unsigned long long) + (size_t)item_tiles(nvox) * 4; }

namespace {
size_t round256(size_t b) { return (b + 255) & ~(size_t)255; }

RayViews ray_views(int nviews, const int32_t *widths, const int32_t *heights) {
    RayViews rv{};
    rv.nviews = nviews;
    for (int v = 0; v < nviews; v++) {
        rv.width[v] = widths[v];
        rv.height[v] = heights[v];
        rv.off[v + 1] = rv.off[v] + (int64_t)widths[v] * heights[v];
        rv.block[v + 1] = rv.block[v] + ((widths[v] + kMarchX - 1) / kMarchX) * ((heights[v] + kMarchY - 1) / kMarchY);
    }
    return rv;
}

// The occupancy grid of the volume into `occ` (occupancy_bytes()).  No grid, so
// that no sample is skipped: without `occ`, and where a sample of zeros would count
// (a negative threshold, an infinite extinction times zero).
OccGrid build_occupancy(hipStream_t s, const uint16_t *vol, int n, float thr, float extinction, void *occ) {
    OccGrid og{nullptr, 1.f, 1.f, 0, 0};
    if (!occ || !(thr >= 0.f) || !std::isfinite(extinction)) return og;
    const int size = (n + 1 + kOccSide - 1) / kOccSide, cells = (n + size) / size;   // lower corners -1 .. n - 1
    // an interpolated value exceeds its corners by a few roundings at most
    const float least = thr * (1.f - 1e-5f);
    const int blocks = (cells + 3) / 4;
    k_occupancy<<<4 * blocks * blocks, 256, 0, s>>>(vol, n, size, cells, least, (uint16_t *)occ);
    og.occ = (const uint2 *)occ;
    og.size = (float)size;
    og.inv_size = 1.f / (float)size;
    og.last = cells - 1;
    og.blocks = blocks;
    return og;
}
}  // namespace

size_t volume_scratch_bytes() { return occupancy_bytes() + sizeof(Selection); }

size_t first_hit_scratch_bytes(int64_t nrays) {
    return round256((size_t)nrays) + 2 * round256((size_t)nrays * 16) +
           256 * sizeof(unsigned long long) + (size_t)item_tiles(nrays) * 4;
}

hipError_t run_first_hits(hipStream_t s, const uint16_t *vol, int n, const gsf_camera *cams,
                          int nviews, const int32_t *widths, const int32_t *heights, float step,
                          float extinction, float thr, float range, const float *lo, const float *hi,
                          float hit_alpha, int color_steps, double opacity, int64_t cap,
                          uint64_t seed, float *params, int64_t *count, int32_t *ray_ids,
                          void *scratch, const VolumeScratch &vs, int cus) {
    if (!vs.device) return hipErrorStreamCaptureUnsupported;   // the call synchronises
    const RayViews rv = ray_views(nviews, widths, heights);
    const int64_t nrays = rv.off[nviews];
    char *sp = (char *)scratch;
    uint8_t *hit = (uint8_t *)sp;
    sp += round256((size_t)nrays);
    float4 *pos = (float4 *)sp;
    sp += round256((size_t)nrays * 16);
    float4 *col = (float4 *)sp;
    sp += round256((size_t)nrays * 16);
    uint32_t *counts = (uint32_t *)(sp + 256 * sizeof(unsigned long long));
    MarchConst mc{};
    mc.n = n;
    mc.color_steps = color_steps;
    mc.step = step;
    mc.extinction = extinction;
    mc.thr = thr;
    mc.inv_range = 1.f / range;
    mc.hit_alpha = hit_alpha;
    for (int c = 0; c < 3; c++) {
        mc.lo[c] = lo[c];
        mc.hi[c] = hi[c];
    }
    const OccGrid og = build_occupancy(s, vol, n, thr, extinction, vs.device);
    k_first_hit<<<rv.block[nviews], kMarchBlock, 0, s>>>(vol, cams, rv, mc, og, hit, pos, col);
    PutHit put{};
    put.pos = pos;
    put.col = col;
    put.P = params;
    put.ray_ids = ray_ids;
    put.log_scale = (float)std::log(2.0 / n);
    put.logit_opacity = (float)std::log(opacity / (1.0 - opacity));
    put.inv_sh_dc = (float)(1.0 / (0.5 / std::sqrt(std::acos(-1.0))));
    return run_select(s, RayItems{hit}, put, nrays, cap, seed, counts, vs, cus, count);
}

hipError_t run_raymarch(hipStream_t s, const uint16_t *vol, int n, const gsf_camera *cams, int nviews,
                        const int32_t *widths, const int32_t *heights, float step, float extinction,
                        float t_stop, float thr, float range, const float *lo, const float *hi,
                        float *out, const VolumeScratch &vs) {
    MarchConst mc{};
    mc.n = n;
    mc.step = step;
    mc.extinction = extinction;
    mc.t_stop = t_stop;
    mc.thr = thr;
    mc.inv_range = 1.f / range;
    for (int c = 0; c < 3; c++) {
        mc.lo[c] = lo[c];
        mc.hi[c] = hi[c];
    }
    const RayViews rv = ray_views(nviews, widths, heights);
    const OccGrid og = build_occupancy(s, vol, n, thr, extinction, vs.device);
    k_raymarch<<<rv.block[nviews], kMarchBlock, 0, s>>>(vol, cams, rv, mc, og, out);
    return hipGetLastError();
}

}  // namespace gsf
