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
// cap-th smallest priority is found by an MSB-first radix select (eight 8-bit
// digit histograms), then the kept voxels are written in raster order.  Mean =
// voxel centre, isotropic log-scale, identity rotation, the given opacity and
// the transfer-function colour as degree-0 SH, in double precision rounded
// once to float.
//
// Ray march: one ray per pixel, emission-absorption through the box
// [-1, 1]^3 in float32 - segments of the step length from the box entry (the
// last shortened to the exit), the trilinear sample (zero outside the grid) at
// each segment's midpoint, density t = clamp((v - thr) / range, 0, 1), colour
// lerp(lo, hi, t), alpha = 1 - exp(-extinction t length), stop once T < t_stop;
// RGB = C + T bg, A = 1 - T.
#include <cmath>
#include <vector>

#include "gs_internal.h"

namespace gsf {
namespace {

constexpr int kVolBlock = 256;
constexpr int kVolIpt = 8;                       // voxels per thread per block
constexpr int kVolTile = kVolBlock * kVolIpt;

__device__ __forceinline__ uint64_t splitmix64(uint64_t state, uint64_t k) {
    uint64_t z = state + k * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__device__ __forceinline__ uint64_t priority(uint64_t seed, uint64_t idx, int ibits) {
    return ((splitmix64(seed, idx + 1ull) >> ibits) << ibits) | idx;
}

// Digit histogram of the candidates whose priority agrees with `prefix` on the
// bits above `shift + 8`; 256 bins accumulated per workgroup in LDS.
__global__ __launch_bounds__(kVolBlock) void k_seed_hist(const uint16_t *__restrict__ vol, int64_t nvox,
                                                         float thr, uint64_t seed, int ibits,
                                                         uint64_t prefix, int shift,
                                                         unsigned long long *__restrict__ hist) {
    __shared__ uint32_t h[256];
    h[threadIdx.x] = 0u;
    __syncthreads();
    const uint64_t hi_mask = shift + 8 >= 64 ? 0ull : ~0ull << (shift + 8);
    for (int64_t i = (int64_t)blockIdx.x * kVolBlock + threadIdx.x; i < nvox;
         i += (int64_t)gridDim.x * kVolBlock) {
        if (!((float)vol[i] > thr)) continue;
        const uint64_t key = priority(seed, (uint64_t)i, ibits);
        if ((key & hi_mask) != (prefix & hi_mask)) continue;
        atomicAdd(&h[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    if (h[threadIdx.x]) atomicAdd(&hist[threadIdx.x], (unsigned long long)h[threadIdx.x]);
}

__device__ __forceinline__ bool kept(const uint16_t *__restrict__ vol, int64_t i, float thr,
                                     uint64_t seed, int ibits, uint64_t kstar) {
    return (float)vol[i] > thr && priority(seed, (uint64_t)i, ibits) <= kstar;
}

// Kept voxels per block of kVolTile voxels.
__global__ __launch_bounds__(kVolBlock) void k_seed_count(const uint16_t *__restrict__ vol, int64_t nvox,
                                                          float thr, uint64_t seed, int ibits,
                                                          uint64_t kstar, uint32_t *__restrict__ counts) {
    __shared__ uint32_t s_cnt;
    if (threadIdx.x == 0) s_cnt = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kVolTile + (int64_t)threadIdx.x * kVolIpt;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kVolIpt; k++)
        if (base + k < nvox && kept(vol, base + k, thr, seed, ibits, kstar)) c++;
    if (c) atomicAdd(&s_cnt, c);
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_cnt;
}

struct SeedConst {
    double inv_n2;          // 2 / n
    double thr, range;
    double lo[3], hi[3];
    double sh_dc;           // value of the constant SH basis function
    float log_scale, logit_opacity;
};

// Writes the kept voxels of its block at offsets[block] + (rank in the block),
// planar [14][m].
__global__ __launch_bounds__(kVolBlock) void k_seed_emit(const uint16_t *__restrict__ vol, int64_t nvox,
                                                         int n, float thr, uint64_t seed, int ibits,
                                                         uint64_t kstar, const uint32_t *__restrict__ offsets,
                                                         SeedConst sc, int64_t m, float *__restrict__ P) {
    __shared__ uint32_t s_wave[kVolBlock / 64];
    const int64_t base = (int64_t)blockIdx.x * kVolTile + (int64_t)threadIdx.x * kVolIpt;
    bool keep[kVolIpt];
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kVolIpt; k++) {
        keep[k] = base + k < nvox && kept(vol, base + k, thr, seed, ibits, kstar);
        c += keep[k] ? 1u : 0u;
    }
    // exclusive scan of c over the block (threads in raster order)
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    uint32_t inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    uint32_t pos = offsets[blockIdx.x] + inc - c;
    for (int k = 0; k < w; k++) pos += s_wave[k];
#pragma unroll
    for (int k = 0; k < kVolIpt; k++) {
        if (!keep[k]) continue;
        const int64_t i = base + k;
        const int64_t ix = i / ((int64_t)n * n), iy = (i / n) % n, iz = i % n;
        const double t0 = ((double)vol[i] - sc.thr) / sc.range;
        const double t = t0 < 0.0 ? 0.0 : (t0 > 1.0 ? 1.0 : t0);
        float *p = P + pos;
        p[0 * m] = (float)(((double)ix + 0.5) * sc.inv_n2 - 1.0);
        p[1 * m] = (float)(((double)iy + 0.5) * sc.inv_n2 - 1.0);
        p[2 * m] = (float)(((double)iz + 0.5) * sc.inv_n2 - 1.0);
        p[3 * m] = p[4 * m] = p[5 * m] = sc.log_scale;
        p[6 * m] = 1.f;
        p[7 * m] = p[8 * m] = p[9 * m] = 0.f;
        p[10 * m] = sc.logit_opacity;
#pragma unroll
        for (int ch = 0; ch < 3; ch++) {
            const double col = sc.lo[ch] * (1.0 - t) + sc.hi[ch] * t;
            p[(11 + ch) * m] = (float)((col - 0.5) / sc.sh_dc);
        }
        pos++;
    }
}

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

// Digit histogram of the hit rays whose priority agrees with `prefix` above `shift`.
__global__ __launch_bounds__(kVolBlock) void k_hit_hist(const uint8_t *__restrict__ hit, int64_t nrays,
                                                        uint64_t seed, int ibits, uint64_t prefix,
                                                        int shift, unsigned long long *__restrict__ hist) {
    __shared__ unsigned long long h[256];
    for (int d = threadIdx.x; d < 256; d += kVolBlock) h[d] = 0ull;
    __syncthreads();
    const uint64_t above = shift >= 56 ? 0ull : (~0ull << (shift + 8));
    for (int64_t i = (int64_t)blockIdx.x * kVolBlock + threadIdx.x; i < nrays;
         i += (int64_t)gridDim.x * kVolBlock) {
        if (!hit[i]) continue;
        const uint64_t key = priority(seed, (uint64_t)i, ibits);
        if ((key & above) != (prefix & above)) continue;
        atomicAdd(&h[(key >> shift) & 0xFFu], 1ull);
    }
    __syncthreads();
    for (int d = threadIdx.x; d < 256; d += kVolBlock)
        if (h[d]) atomicAdd(&hist[d], h[d]);
}

__device__ __forceinline__ bool hit_kept(const uint8_t *hit, int64_t i, uint64_t seed, int ibits,
                                         uint64_t kstar) {
    return hit[i] && priority(seed, (uint64_t)i, ibits) <= kstar;
}

// Kept rays per block of kVolTile rays.
__global__ __launch_bounds__(kVolBlock) void k_hit_count(const uint8_t *__restrict__ hit, int64_t nrays,
                                                         uint64_t seed, int ibits, uint64_t kstar,
                                                         uint32_t *__restrict__ counts) {
    __shared__ uint32_t s_c;
    if (threadIdx.x == 0) s_c = 0u;
    __syncthreads();
    const int64_t base = (int64_t)blockIdx.x * kVolTile + (int64_t)threadIdx.x * kVolIpt;
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kVolIpt; k++) c += base + k < nrays && hit_kept(hit, base + k, seed, ibits, kstar) ? 1u : 0u;
    if (c) atomicAdd(&s_c, c);
    __syncthreads();
    if (threadIdx.x == 0) counts[blockIdx.x] = s_c;
}

struct HitEmit {
    float log_scale, logit_opacity, inv_sh_dc;
};

// Gaussians of the kept rays, in ray order, planar [14][m]; ray_ids nullable.
__global__ __launch_bounds__(kVolBlock) void k_hit_emit(const uint8_t *__restrict__ hit, int64_t nrays,
                                                        uint64_t seed, int ibits, uint64_t kstar,
                                                        const uint32_t *__restrict__ offsets,
                                                        const float4 *__restrict__ pos,
                                                        const float4 *__restrict__ col, HitEmit he,
                                                        int64_t m, float *__restrict__ P,
                                                        int32_t *__restrict__ ray_ids) {
    __shared__ uint32_t s_wave[kVolBlock / 64];
    const int64_t base = (int64_t)blockIdx.x * kVolTile + (int64_t)threadIdx.x * kVolIpt;
    bool keep[kVolIpt];
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kVolIpt; k++) {
        keep[k] = base + k < nrays && hit_kept(hit, base + k, seed, ibits, kstar);
        c += keep[k] ? 1u : 0u;
    }
    const int lane = __lane_id(), w = threadIdx.x >> 6;
    uint32_t inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(inc, o, 64);
        if (lane >= o) inc += y;
    }
    if (lane == 63) s_wave[w] = inc;
    __syncthreads();
    uint32_t at = offsets[blockIdx.x] + inc - c;
    for (int k = 0; k < w; k++) at += s_wave[k];
#pragma unroll
    for (int k = 0; k < kVolIpt; k++) {
        if (!keep[k]) continue;
        const int64_t i = base + k;
        const float4 p4 = pos[i], c4 = col[i];
        float *p = P + at;
        p[0 * m] = p4.x;
        p[1 * m] = p4.y;
        p[2 * m] = p4.z;
        p[3 * m] = p[4 * m] = p[5 * m] = he.log_scale;
        p[6 * m] = 1.f;
        p[7 * m] = p[8 * m] = p[9 * m] = 0.f;
        p[10 * m] = he.logit_opacity;
        p[11 * m] = (c4.x - 0.5f) * he.inv_sh_dc;
        p[12 * m] = (c4.y - 0.5f) * he.inv_sh_dc;
        p[13 * m] = (c4.z - 0.5f) * he.inv_sh_dc;
        if (ray_ids) ray_ids[at] = (int32_t)i;
        at++;
    }
}

}  // namespace

int seed_blocks(int64_t nvox) { return (int)((nvox + kVolTile - 1) / kVolTile); }

// Host side of the seeding (synchronises the stream several times).
hipError_t run_seed(hipStream_t s, const uint16_t *vol, int n, double thr, double range,
                    const double *lo, const double *hi, double opacity, int64_t cap, uint64_t seed,
                    float *params, int64_t *count, void *scratch) {
    const int64_t nvox = (int64_t)n * n * n;
    int ibits = 0;
    while ((int64_t(1) << ibits) < nvox) ibits++;
    if (ibits < 1) ibits = 1;
    unsigned long long *hist = (unsigned long long *)scratch;                 // 256
    uint32_t *counts = (uint32_t *)((char *)scratch + 256 * sizeof(unsigned long long));
    const int nb = seed_blocks(nvox);
    std::vector<unsigned long long> h(256);
    std::vector<uint32_t> cnt(nb);
    int grid = nb < 1024 ? nb : 1024;
    // MSB-first radix select of the cap-th smallest priority among the candidates
    uint64_t prefix = 0;
    int64_t rank = cap;          // 1-based rank still to find within the prefix
    int64_t total = -1;
    for (int shift = 56; shift >= 0; shift -= 8) {
        hipError_t e = hipMemsetAsync(hist, 0, 256 * sizeof(unsigned long long), s);
        if (e != hipSuccess) return e;
        k_seed_hist<<<grid, kVolBlock, 0, s>>>(vol, nvox, (float)thr, seed, ibits, prefix, shift, hist);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = hipMemcpyAsync(h.data(), hist, 256 * sizeof(unsigned long long), hipMemcpyDeviceToHost, s)) != hipSuccess)
            return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (total < 0) {
            total = 0;
            for (int d = 0; d < 256; d++) total += (int64_t)h[d];
            if (total <= cap) {     // every candidate is kept
                prefix = ~0ull;
                rank = 0;
                break;
            }
        }
        int d = 0;
        while (d < 255 && (int64_t)h[d] < rank) rank -= (int64_t)h[d++];
        prefix |= (uint64_t)d << shift;
    }
    const uint64_t kstar = prefix;   // priorities are distinct: exactly min(total, cap) are <= kstar
    k_seed_count<<<nb, kVolBlock, 0, s>>>(vol, nvox, (float)thr, seed, ibits, kstar, counts);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if ((e = hipMemcpyAsync(cnt.data(), counts, nb * sizeof(uint32_t), hipMemcpyDeviceToHost, s)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    int64_t m = 0;
    for (int b = 0; b < nb; b++) {
        const uint32_t c = cnt[b];
        cnt[b] = (uint32_t)m;
        m += c;
    }
    if ((e = hipMemcpyAsync(counts, cnt.data(), nb * sizeof(uint32_t), hipMemcpyHostToDevice, s)) != hipSuccess)
        return e;
    SeedConst sc;
    sc.inv_n2 = 2.0 / n;
    sc.thr = thr;
    sc.range = range;
    for (int c = 0; c < 3; c++) {
        sc.lo[c] = lo[c];
        sc.hi[c] = hi[c];
    }
    sc.sh_dc = 0.5 / std::sqrt(std::acos(-1.0));
    sc.log_scale = (float)std::log(2.0 / n);
    sc.logit_opacity = (float)std::log(opacity / (1.0 - opacity));
    k_seed_emit<<<nb, kVolBlock, 0, s>>>(vol, nvox, n, (float)thr, seed, ibits, kstar, counts, sc, m, params);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    *count = m;
    return hipSuccess;
}

size_t seed_scratch_bytes(int64_t nvox) { return 256 * sizeof(unsigned long long) + (size_t)seed_blocks(nvox) * 4; }

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

size_t occupancy_bytes() { return (size_t)kOccSide * kOccSide * kOccSide / 8; }

size_t first_hit_scratch_bytes(int64_t nrays) {
    return round256((size_t)nrays) + 2 * round256((size_t)nrays * 16) +
           256 * sizeof(unsigned long long) + (size_t)seed_blocks(nrays) * 4;
}

hipError_t run_first_hits(hipStream_t s, const uint16_t *vol, int n, const gsf_camera *cams,
                          int nviews, const int32_t *widths, const int32_t *heights, float step,
                          float extinction, float thr, float range, const float *lo, const float *hi,
                          float hit_alpha, int color_steps, double opacity, int64_t cap,
                          uint64_t seed, float *params, int64_t *count, int32_t *ray_ids,
                          void *scratch, void *occ) {
    const RayViews rv = ray_views(nviews, widths, heights);
    const int64_t nrays = rv.off[nviews];
    char *sp = (char *)scratch;
    uint8_t *hit = (uint8_t *)sp;
    sp += round256((size_t)nrays);
    float4 *pos = (float4 *)sp;
    sp += round256((size_t)nrays * 16);
    float4 *col = (float4 *)sp;
    sp += round256((size_t)nrays * 16);
    unsigned long long *hist = (unsigned long long *)sp;
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
    const OccGrid og = build_occupancy(s, vol, n, thr, extinction, occ);
    k_first_hit<<<rv.block[nviews], kMarchBlock, 0, s>>>(vol, cams, rv, mc, og, hit, pos, col);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    int ibits = 0;
    while ((int64_t(1) << ibits) < nrays) ibits++;
    if (ibits < 1) ibits = 1;
    const int nb = seed_blocks(nrays);
    std::vector<unsigned long long> h(256);
    std::vector<uint32_t> cnt(nb);
    const int grid = nb < 1024 ? nb : 1024;
    // MSB-first radix select of the cap-th smallest priority among the hit rays
    uint64_t prefix = 0;
    int64_t rank = cap;
    int64_t total = -1;
    for (int shift = 56; shift >= 0; shift -= 8) {
        if ((e = hipMemsetAsync(hist, 0, 256 * sizeof(unsigned long long), s)) != hipSuccess) return e;
        k_hit_hist<<<grid, kVolBlock, 0, s>>>(hit, nrays, seed, ibits, prefix, shift, hist);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        if ((e = hipMemcpyAsync(h.data(), hist, 256 * sizeof(unsigned long long), hipMemcpyDeviceToHost, s)) != hipSuccess)
            return e;
        if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
        if (total < 0) {
            total = 0;
            for (int d = 0; d < 256; d++) total += (int64_t)h[d];
            if (total <= cap) {     // every hit is kept
                prefix = ~0ull;
                break;
            }
        }
        int d = 0;
        while (d < 255 && (int64_t)h[d] < rank) rank -= (int64_t)h[d++];
        prefix |= (uint64_t)d << shift;
    }
    const uint64_t kstar = prefix;   // priorities are distinct: min(total, cap) are <= kstar
    k_hit_count<<<nb, kVolBlock, 0, s>>>(hit, nrays, seed, ibits, kstar, counts);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipMemcpyAsync(cnt.data(), counts, nb * sizeof(uint32_t), hipMemcpyDeviceToHost, s)) != hipSuccess)
        return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    int64_t m = 0;
    for (int b = 0; b < nb; b++) {
        const uint32_t c = cnt[b];
        cnt[b] = (uint32_t)m;
        m += c;
    }
    if ((e = hipMemcpyAsync(counts, cnt.data(), nb * sizeof(uint32_t), hipMemcpyHostToDevice, s)) != hipSuccess)
        return e;
    HitEmit he;
    he.log_scale = (float)std::log(2.0 / n);
    he.logit_opacity = (float)std::log(opacity / (1.0 - opacity));
    he.inv_sh_dc = (float)(1.0 / (0.5 / std::sqrt(std::acos(-1.0))));
    k_hit_emit<<<nb, kVolBlock, 0, s>>>(hit, nrays, seed, ibits, kstar, counts, pos, col, he, m,
                                       params, ray_ids);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    if ((e = hipStreamSynchronize(s)) != hipSuccess) return e;
    *count = m;
    return hipSuccess;
}

hipError_t run_raymarch(hipStream_t s, const uint16_t *vol, int n, const gsf_camera *cams, int nviews,
                        const int32_t *widths, const int32_t *heights, float step, float extinction,
                        float t_stop, float thr, float range, const float *lo, const float *hi,
                        float *out, void *occ) {
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
    const OccGrid og = build_occupancy(s, vol, n, thr, extinction, occ);
    k_raymarch<<<rv.block[nviews], kMarchBlock, 0, s>>>(vol, cams, rv, mc, og, out);
    return hipGetLastError();
}

}  // namespace gsf
