// raster.hip - per-tile front-to-back alpha compositing, its back-to-front
// adjoint, and the masked L1 image loss.
//
// One workgroup per screen tile (T x T pixels, T in {8, 16, 32}); one thread
// per pixel (T = 32: four pixels per thread).  The tile's depth-ordered list of
// splats is staged through LDS in batches of B records (B in {64, 128, 256})
// that every wave then reads by broadcast.  Per pixel and splat, with the
// projection's conic pre-scaled by log2(e) so that power2 = log2(e) * power:
//   skip if power2 > 0 or power2 < tau, tau = log2(1 / (255 o))
//        (the second test is o e^power < 1/255 without the exponential);
//   alpha = min(0.99, o 2^power2);
//   stop before the splat if T (1 - alpha) < 1e-4;
//   C += colour alpha T;  T *= 1 - alpha.
// A wave leaves the batch once all its pixels have stopped (checked every four
// splats) and the workgroup leaves the tile once all waves have.  A pixel's
// arithmetic sequence does not depend on T, B or the tile's other pixels, so
// images are bitwise independent of the tile size and the batch size.
//
// The adjoint walks the same list back to front from each pixel's last
// included splat.  Transmittance modes: recompute (the transmittance in front
// of each splat is rebuilt as T_i = T_{i+1} / (1 - alpha_i) from the final
// state; one workgroup per tile), checkpointed ((T, colour) stored by the
// forward at every LDS-batch boundary; persistent workgroups over (tile, batch)
// units, each rebuilding T within its batch) and stored (the forward stores
// T_i of every included (splat, pixel) pair at [key position][pixel of tile];
// the adjoint reads it; one workgroup per tile).  The nine per-splat screen-space
// gradient terms are summed over a tile's pixels and stored once per (key, field)
// at the key's own position; a separate pass sums each record's keys (no atomics).
// Two forms of the adjoint: for plans of few tiles one wave per 8x8 block, which sums
// the terms of eight splats with matrix products (more waves than tiles); for many
// tiles one wave per tile, which folds them with DPP adds and LDS rows (fewer vector
// cycles).  Where a wave covers an 8x8 quadrant of a 16-pixel tile it skips the splats
// whose padded support ellipse misses it.
#include <type_traits>

#include "gs_internal.h"

namespace gsf {
namespace {

constexpr float kLn2 = 0.69314718055994531f;

// Shared by every kernel that walks a tile list so all take identical decisions.
// a = (hx, hy, A2, B2), b = (C2, opacity, red, green), c = (blue, limit, ix, iy)
// with A2 = -log2(e) A / 2, B2 = -log2(e) B, C2 = -log2(e) C / 2; (x, y) is
// the integer pixel (as float) and (dx, dy) its centre's offset from the mean.
__device__ __forceinline__ float splat_dx(float x, float ix, float hx) { return (x - ix) + hx; }

// -power2 = -(A2 dx^2 + B2 dx dy + C2 dy^2), evaluated as -(dx (A2 dx + B2 dy) + (C2 dy) dy)
// (five operations, the signs being modifiers); every kernel that decides inclusion
// uses this one form.
__device__ __forceinline__ float splat_fall(const float4 &a, const float4 &b, float dx, float dy) {
    return fmaf(-dx, fmaf(a.z, dx, a.w * dy), ((-b.x) * dy) * dy);
}
// Whether a splat with this fall is included: 0 <= fall <= -tau, one comparison of
// the bits with the record's limit, the bits of -tau plus one (a negative fall has the
// sign bit; it is never -0, as (-C2 dy) dy is at least +0).
__device__ __forceinline__ bool splat_within(float fall, float limit) {
    return __float_as_uint(fall) < __float_as_uint(limit);
}

__device__ __forceinline__ bool splat_alpha(const float4 &a, const float4 &b, const float4 &c,
                                            float x, float y, float &alpha, float &ae, float &ex,
                                            float &dx, float &dy) {
    dx = splat_dx(x, c.z, a.x);
    dy = splat_dx(y, c.w, a.y);
    const float fall = splat_fall(a, b, dx, dy);
    if (!splat_within(fall, c.y)) return false;
    ex = __builtin_amdgcn_exp2f(-fall);
    ae = b.y * ex;
    alpha = fminf(kAlphaMax, ae);
    return true;
}

// A record's c = (blue, limit, ix, iy): the limit comes of tau = -log2(255 o), the
// alpha threshold of the base-2 exponent, computed once by the projection.  The
// padded half height of the support (where o e^power >= 1/255 can hold) is
// the ellipse's y extent plus the absolute padding.
// Half height of the padded ellipse for the quadrant test, with the hardware
// reciprocal and square root: their few-ulp error lies far inside the padding,
// and the forward and the adjoint both use this form, so they skip the same
// quadrants.  (Tile enumeration keeps the exact form everywhere.)
__device__ __forceinline__ float quad_half_height(const float4 &e0) {
    return __builtin_amdgcn_sqrtf(e0.y * __builtin_amdgcn_rcpf(e0.z));
}

typedef __attribute__((address_space(3))) void *lds_void_ptr;
__device__ __forceinline__ lds_void_ptr lds_ptr(void *p) { return (lds_void_ptr)p; }

__device__ __forceinline__ int view_of_tile(const ViewDesc *__restrict__ views, int nviews, int gt) {
    int v = 0;
    while (v + 1 < nviews && gt >= views[v + 1].tile_off) v++;
    return v;
}

// Launch tile c of the compositing kernels: a global tile id, or (tm.gaze) a
// compact fovea-box id (view c / box^2, then row-major from the view's first
// fovea tile, as the fovea-culled sort keys).  False for a box tile past the
// view's fovea tiles (no pixel of it is composited).
__device__ __forceinline__ bool launch_tile(uint32_t c, const TileMap &tm,
                                            const ViewDesc *__restrict__ views, int nviews, int T,
                                            int &v, ViewDesc &vd, int &ty, int &tx) {
    if (tm.gaze) {
        const uint32_t box = (uint32_t)tm.box, area = box * box;
        v = (int)(c / area);
        const uint32_t l = c - (uint32_t)v * area, ly = l / box;
        vd = views[v];
        const FoveaTiles f = fovea_tiles(tm.gaze, v, tm.radius, vd.width, vd.height, T);
        ty = f.ty0 + (int)ly;
        tx = f.tx0 + (int)(l - ly * box);
        return tx <= f.tx1 && ty <= f.ty1;
    }
    v = view_of_tile(views, nviews, (int)c);
    vd = views[v];
    const int local = (int)c - vd.tile_off;
    ty = local / vd.tiles_x;
    tx = local - ty * vd.tiles_x;
    return true;
}

// Pixel (x, y) of view v lies in the fovea disk (the loss's mask): its centre
// within `radius` pixels of the gaze point, tested in FP32; no gaze: every pixel.
__device__ __forceinline__ bool in_fovea(const float *__restrict__ gaze, int v, int x, int y,
                                         float radius) {
    if (!gaze) return true;
    const float dx = (float)x + 0.5f - gaze[2 * v], dy = (float)y + 0.5f - gaze[2 * v + 1];
    return dx * dx + dy * dy <= radius * radius;
}

// MODE 1 (checkpointed): also store (T, colour) of every pixel after each LDS
// batch that is not the tile's last (slot = boundary position / B, unique over
// all tiles) and the final (T, colour), so the adjoint can start at any batch.
// MODE 2 (stored): also store T in front of every included pair at
// tstore[key position * T*T + pixel of tile].
// One workgroup per tile, workgroup i taking tile order[i]: the order lists
// tiles with more keys first, so the dispatcher starts the heavy tiles on
// different CUs at once and fills in with light ones as slots free up, however
// the keys cluster on screen.
// Threads of a forward workgroup: one per pixel (at most 256).  A 16-pixel
// tile is composited by four waves, one per 8x8 quadrant, each skipping the
// splats whose padded ellipse misses its quadrant.  SPLIT (16-pixel tiles):
// the four quadrants are four one-wave workgroups instead; they run
// independently, each with no barrier shared with the others, at the cost of
// staging every batch four times, which pays only where the heaviest tiles,
// not throughput, set the time (few tiles; the launcher's choice).
// Workgroups are dealt to the 8 XCDs round robin (workgroup g to XCD g mod
// 8), so workgroup g takes quadrant (g >> 3) & 3 of the tile at position
// 8 (g >> 5) + (g & 7) of the order: the four quadrants of a tile share an
// XCD and its L2, and the order's heaviest tiles still come first.
template <int T, bool SPLIT>
constexpr int fwd_threads() { return SPLIT ? 64 : (T * T < 256 ? T * T : 256); }

template <int T, int B, int MODE, bool SPLIT>
__global__ __launch_bounds__((fwd_threads<T, SPLIT>())) void k_render_fwd(
    const uint32_t *__restrict__ order,
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ vals, SplatPtrs sp,
    const ViewDesc *__restrict__ views, int nviews, const gsf_camera *__restrict__ cams,
    float *__restrict__ out_rgba, float *__restrict__ tfinal, uint32_t *__restrict__ ncontrib,
    float4 *__restrict__ ckpt, float4 *__restrict__ fstate, float *__restrict__ tstore,
    const float *__restrict__ bg, const float *__restrict__ cull_gaze, float cull_radius,
    int total_tiles, TileMap tm) {
    constexpr bool CKPT = MODE == 1;
    constexpr bool QUAD = T == 16;   // a wave composites one 8 x 8 quadrant
    static_assert(!SPLIT || QUAD, "only 16-pixel tiles are split");
    constexpr int NT = fwd_threads<T, SPLIT>();
    constexpr int PPT = QUAD ? 1 : T * T / NT;
    constexpr int ROWS = NT / T;
    constexpr int U = 4;   // splats between wave-level completion checks
    static_assert(U == 4, "a group of splat indices is read as one int4");
    // AHEAD (split tiles, whose few waves cannot hide the LDS reads): the reads of
    // a group are issued before the group in front of it is blended, two sets of
    // registers in turn (4% on one view of 1024^2, 5% on one of 512^2).
    constexpr bool AHEAD = SPLIT;
    constexpr int kPad = AHEAD ? 4 * U : U;
    constexpr int kListLen = 64 + kPad;   // per wave: one 64-splat chunk, padded
    // PREF (a batch no larger than the workgroup): two LDS buffers; the
    // records of the next batch are copied from global memory straight into
    // the other buffer (global_load_lds, no registers; wave w copies entries
    // 64 w .. 64 w + 63) while the current batch composites, the record ids
    // being read one batch further ahead.
    constexpr bool PREF = B <= NT;
    // A buffer holds the batch's records a, b, c and support ellipses
    // (slope, kw, ws, dyr) at sections 0, 1, 2, 3 of B + 1 entries.  Buffers
    // 0 and 1 are separate arrays, so the compiler sees that reads of one do
    // not wait for copies into the other.  Entry B of a, b, c: an inert splat
    // (limit 0: never included) that pads a wave's last
    // group of U.
    // (Entry 0 of each array is unused: a copy addressed at an array's very
    // start loses the alias information that lets reads of the other buffer
    // proceed while it is in flight.)
    constexpr int SEC = B + 1;
    constexpr int NW = NT / 64;
    __shared__ __align__(16) int s_list[NW * kListLen];
    // the waves' votes of a workgroup-wide test, two rows used in turn: a row is
    // written again only two votes later, after a barrier that every wave
    // reaches once it has read the row
    __shared__ __align__(16) uint32_t s_vote[2][NW < 4 ? 4 : NW];
    __shared__ float4 s_buf0_[1 + 4 * SEC];
    __shared__ float4 s_buf1_[PREF ? 1 + 4 * SEC : 1];
    float4 *const s_buf0 = s_buf0_ + 1;
    float4 *const s_buf1 = s_buf1_ + 1;

    const int quad = SPLIT ? (int)((blockIdx.x >> 3) & 3u) : (int)(threadIdx.x >> 6);
    const uint32_t oi = SPLIT ? (blockIdx.x >> 5) * 8u + (blockIdx.x & 7u) : blockIdx.x;
    if (oi >= (uint32_t)total_tiles) return;   // the split grid is padded to whole groups of 8 tiles
    const uint32_t ti = order[oi];
    int v, ty, tx;
    ViewDesc vd;
    if (!launch_tile(ti, tm, views, nviews, T, v, vd, ty, tx)) return;
    // Fovea culling: only the pixels of the fovea disk are composited; the others,
    // which carry no loss, start stopped (background, no contributor).  Over the
    // compact fovea-box tiles, a tile that cannot hold a pixel of the disk is not
    // visited at all (the adjoint skips it alike); over global tiles every tile
    // is, so that each holds its pixels' state.
    if (tm.gaze && !fovea_tile_live(tm.gaze, v, tm.radius, vd.width, vd.height, T, tx, ty)) return;
    const float disk_r = cull_gaze ? cull_radius * (float)vd.width : 0.f;
    const uint2 rg = ranges[ti];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int lx = QUAD ? (quad & 1) * 8 + (lane & 7) : threadIdx.x % T;
    const int ly = QUAD ? (quad >> 1) * 8 + (lane >> 3) : threadIdx.x / T;
    if (threadIdx.x == 0) {
        s_buf0[B] = make_float4(0.f, 0.f, 0.f, 0.f);
        s_buf0[SEC + B] = make_float4(0.f, 0.f, 0.f, 0.f);
        s_buf0[2 * SEC + B] = make_float4(0.f, 0.f, 0.f, 0.f);
        if constexpr (PREF) {
            s_buf1[B] = make_float4(0.f, 0.f, 0.f, 0.f);
            s_buf1[SEC + B] = make_float4(0.f, 0.f, 0.f, 0.f);
            s_buf1[2 * SEC + B] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
    }

    // Whether `pred` holds on every thread of the workgroup: one barrier (the
    // waves' votes in LDS), which also ends the batch's copies into LDS and its
    // reads of the buffer.
    uint32_t vrow = 0u;
    auto block_all = [&](bool pred) -> bool {
        const bool w = __all(pred);
        if constexpr (NW == 1) {
            __syncthreads();
            return w;
        } else {
            if (lane == 0) s_vote[vrow][wave] = w ? 1u : 0u;
            __syncthreads();
            uint32_t r = 1u;
#pragma unroll
            for (int i = 0; i < NW; i++) r &= s_vote[vrow][i];
            vrow ^= 1u;
            return r != 0u;
        }
    };

    // Tr[k] is the pixel's transmittance while it composites; a pixel that has
    // stopped (or lies outside the image) holds -T instead, so one compare
    // gives its state and no flag is carried from splat to splat.
    float px[PPT], py[PPT], Tr[PPT], cr[PPT], cg[PPT], cb[PPT];
    uint32_t last[PPT];
    int pix[PPT];   // the pixel's row-major index in the tile
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int x = tx * T + lx, y = ty * T + ly + k * ROWS;
        px[k] = (float)x;   // integer pixel; its centre's offset from a mean is splat_dx
        py[k] = (float)y;
        pix[k] = (ly + k * ROWS) * T + lx;
        Tr[k] = x < vd.width && y < vd.height && in_fovea(cull_gaze, v, x, y, disk_r) ? 1.f : -1.f;
        cr[k] = cg[k] = cb[k] = 0.f;
        last[k] = 0u;
    }

    // Composite the batch at bs from one LDS buffer; true once every pixel of
    // the tile has stopped.  Ends with a barrier, after which the buffer is free.
    auto composite = [&](uint32_t bs, const float4 *buf) -> bool {
        const float4 *SA = buf, *SB = buf + SEC, *SC = buf + 2 * SEC, *SE = buf + 3 * SEC;
        const int nb = (int)min((uint32_t)B, rg.y - bs);
        // list entries are the byte offset 16 j of the splat's slot j in a
        // section, which the LDS reads take as their address (the section's
        // start being the constant part); slot j is the splat's 1-based place
        // j + off in the tile's list, what last[] records: within the batch the
        // pixel keeps the offset (lastb, ~0 for none) and converts it at the end
        const int off = (int)(bs - rg.x) + 1;
        uint32_t lastb[PPT];
#pragma unroll
        for (int k = 0; k < PPT; k++) lastb[k] = ~0u;
        // a wave whose pixels have all stopped (or start outside the disk or
        // the image) skips the batch: no quadrant tests, no list
        bool stopped = true;
#pragma unroll
        for (int k = 0; k < PPT; k++) stopped &= !(Tr[k] > 0.f);
        bool done = __all(stopped);
        // the batch 64 splats at a time: the wave's splats are the set bits of
        // m (with 16-pixel tiles, those whose padded ellipse reaches the wave's
        // quadrant)
        for (int cb0 = 0; cb0 < nb && !done; cb0 += 64) {
            const int jl = cb0 + lane;
            bool meet = jl < nb;
            if (QUAD && meet) {
                const float4 e0 = SE[jl], a0 = SA[jl], c0 = SC[jl];
                const Ellipse e{e0.x, e0.y, e0.z, e0.w, quad_half_height(e0), a0.x, a0.y, (int)c0.z, (int)c0.w};
                meet = quad_meets(e, tx * T + (quad & 1) * 8, ty * T + (quad >> 1) * 8);
            }
            // the wave's list of them in LDS, padded with the inert slot to whole
            // groups of U, read back a group at a time (the indices stay in
            // vector registers: no scalar bookkeeping per splat)
            const uint64_t m = __ballot(meet);
            const int cnt = (int)__popcll(m);
            int *list = s_list + wave * kListLen;
            if (meet) list[lanes_below(m)] = jl * (int)sizeof(float4);
            if (lane < kPad) list[cnt + lane] = B * (int)sizeof(float4);
            struct Group {
                uint32_t bo[U];
                float4 a[U], b[U], c[U];
            };
            auto read_group = [&](const int4 &j4) __attribute__((always_inline)) {
                Group q;
                q.bo[0] = (uint32_t)j4.x;
                q.bo[1] = (uint32_t)j4.y;
                q.bo[2] = (uint32_t)j4.z;
                q.bo[3] = (uint32_t)j4.w;
#pragma unroll
                for (int u = 0; u < U; u++) {
                    q.a[u] = *(const float4 *)((const char *)SA + q.bo[u]);
                    q.b[u] = *(const float4 *)((const char *)SB + q.bo[u]);
                    q.c[u] = *(const float4 *)((const char *)SC + q.bo[u]);
                }
                return q;
            };
            auto all_stopped = [&]() __attribute__((always_inline)) {
                bool all = true;
#pragma unroll
                for (int k = 0; k < PPT; k++) all &= !(Tr[k] > 0.f);
                return (bool)__all(all);
            };
            auto blend = [&](const Group &q) __attribute__((always_inline)) {
                const uint32_t(&bo)[U] = q.bo;
                const float4(&a)[U] = q.a, (&b)[U] = q.b, (&c)[U] = q.c;
#pragma unroll
                for (int k = 0; k < PPT; k++) {
                    float alpha[U];
                    bool valid[U];
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        const float dx = splat_dx(px[k], c[u].z, a[u].x);
                        const float dy = splat_dx(py[k], c[u].w, a[u].y);
                        const float fall = splat_fall(a[u], b[u], dx, dy);
                        valid[u] = splat_within(fall, c[u].y);
                        alpha[u] = valid[u] ? fminf(kAlphaMax, b[u].y * __builtin_amdgcn_exp2f(-fall)) : 0.f;
                    }
                    // Phase 2: the sequential front-to-back update.  An included
                    // splat performs exactly the float operations of the definition
                    // (Tn = T (1 - alpha), w = alpha T, C += colour w); any other
                    // has alpha 0, or gets w = 0, which leaves T and the
                    // (non-negative) colour sums as they are bit for bit.  That the
                    // skipped ones are folded into alpha in phase 1 keeps scalar
                    // mask operations off the chain from T to T (5 to 7% of the
                    // kernel, 11% where a wave has a SIMD for itself; what bounds it is the
                    // 24 vector operations a splat and pixel, 72 cycles).  Branches
                    // around the update instead of selects: 5 to 10% slower; a form
                    // without the stop test for groups in which no pixel stops: 4 to 7%.
#pragma unroll
                    for (int u = 0; u < U; u++) {
                        // A stopped pixel holds -T < 0, so its Tn < 0 < kTStop: it is
                        // never included, and -|T| keeps it stopped.  A running pixel
                        // stops where Tn < kTStop and then holds -T.
                        const float Tn = Tr[k] * (1.f - alpha[u]);
                        const bool on = !(Tn < kTStop);
                        if (MODE == 2 && valid[u] && on)
                            tstore[(size_t)(bs + bo[u] / (uint32_t)sizeof(float4)) * (T * T) + pix[k]] = Tr[k];
                        const float w = (on ? alpha[u] : 0.f) * Tr[k];
                        cr[k] = fmaf(b[u].z, w, cr[k]);
                        cg[k] = fmaf(b[u].w, w, cg[k]);
                        cb[k] = fmaf(c[u].x, w, cb[k]);
                        Tr[k] = on ? Tn : -fabsf(Tr[k]);
                        lastb[k] = valid[u] && on ? bo[u] : lastb[k];
                    }
                }
            };
            if constexpr (AHEAD) {
                Group q0 = read_group(*(const int4 *)list), q1;
                int4 j = *(const int4 *)(list + U);
                for (int g = 0; g < cnt; g += 2 * U) {
                    if (all_stopped()) {
                        done = true;
                        break;
                    }
                    q1 = read_group(j);
                    j = *(const int4 *)(list + g + 2 * U);
                    blend(q0);
                    if (g + U >= cnt) break;
                    if (all_stopped()) {
                        done = true;
                        break;
                    }
                    q0 = read_group(j);
                    j = *(const int4 *)(list + g + 3 * U);
                    blend(q1);
                }
            } else {
                for (int g = 0; g < cnt; g += U) {
                    if (all_stopped()) {
                        done = true;
                        break;
                    }
                    blend(read_group(*(const int4 *)(list + g)));
                }
            }
        }
#pragma unroll
        for (int k = 0; k < PPT; k++)
            if (lastb[k] != ~0u) last[k] = lastb[k] / (uint32_t)sizeof(float4) + (uint32_t)off;
        if (CKPT && bs + B < rg.y) {
            float4 *slot = ckpt + (size_t)((bs + B) / B) * (T * T);
#pragma unroll
            for (int k = 0; k < PPT; k++)
                slot[pix[k]] = make_float4(fabsf(Tr[k]), cr[k], cg[k], cb[k]);
        }
        bool all = true;
#pragma unroll
        for (int k = 0; k < PPT; k++) all &= !(Tr[k] > 0.f);
        return block_all(all);
    };

    // A workgroup none of whose pixels composites (all outside the fovea disk or
    // the image) stages nothing: its pixels are written as they start.
    bool any_px = false;
#pragma unroll
    for (int k = 0; k < PPT; k++) any_px |= Tr[k] > 0.f;
    if (!block_all(!any_px)) {
        if constexpr (PREF) {
            // copy record r of entry threadIdx.x into a buffer (this wave's 64 slots)
            auto stage = [&](float4 *buf, uint32_t r) {
                float4 *d = buf + (threadIdx.x & ~63u);
                const float4 *rr = sp.at(r, 0);   // one 64-byte chunk: a, b, c, ellipse
                __builtin_amdgcn_global_load_lds((const void *)(rr + kRecA), lds_ptr(d), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((const void *)(rr + kRecB), lds_ptr(d + SEC), 16, 0, 0);
                __builtin_amdgcn_global_load_lds((const void *)(rr + kRecC), lds_ptr(d + 2 * SEC), 16, 0, 0);
                if constexpr (QUAD)
                    __builtin_amdgcn_global_load_lds((const void *)(rr + kRecEll), lds_ptr(d + 3 * SEC), 16, 0, 0);
            };
            const uint32_t j = threadIdx.x;
            uint32_t rnext = 0u;
            if (j < (uint32_t)B && rg.x + j < rg.y) stage(s_buf0, vals[rg.x + j]);
            if (j < (uint32_t)B && rg.x + B + j < rg.y) rnext = vals[rg.x + B + j];
            __syncthreads();   // the inert slots and the first batch
            // Batches alternate between the buffers.  A batch has arrived before
            // the barrier that ended the previous one, after which the other
            // buffer is free: the next batch is copied there while this one
            // composites.
            for (uint32_t bs = rg.x; bs < rg.y;) {
                if (j < (uint32_t)B && bs + B + j < rg.y) stage(s_buf1, rnext);
                if (j < (uint32_t)B && bs + 2 * B + j < rg.y) rnext = vals[bs + 2 * B + j];
                if (composite(bs, s_buf0)) break;
                if ((bs += B) >= rg.y) break;
                if (j < (uint32_t)B && bs + B + j < rg.y) stage(s_buf0, rnext);
                if (j < (uint32_t)B && bs + 2 * B + j < rg.y) rnext = vals[bs + 2 * B + j];
                if (composite(bs, s_buf1)) break;
                bs += B;
            }
        } else {
            __syncthreads();   // the inert slots
            for (uint32_t bs = rg.x; bs < rg.y; bs += B) {
                const int nb = (int)min((uint32_t)B, rg.y - bs);
                for (int j = threadIdx.x; j < nb; j += NT) {
                    const float4 *rr = sp.at(vals[bs + j], 0);
                    s_buf0[j] = rr[kRecA];
                    s_buf0[SEC + j] = rr[kRecB];
                    s_buf0[2 * SEC + j] = rr[kRecC];
                    if constexpr (QUAD) s_buf0[3 * SEC + j] = rr[kRecEll];
                }
                __syncthreads();
                if (composite(bs, s_buf0)) break;
            }
        }
    }
#pragma unroll
    for (int k = 0; k < PPT; k++) Tr[k] = fabsf(Tr[k]);

    const float *bgv = bg ? bg + 3 * v : cams[v].bg;
    const float bg0 = bgv[0], bg1 = bgv[1], bg2 = bgv[2];
    const size_t plane = (size_t)vd.width * vd.height;
    float *img = out_rgba + 4 * (size_t)vd.pix_off;
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int x = tx * T + lx, y = ty * T + ly + k * ROWS;
        if (!(x < vd.width && y < vd.height)) continue;
        const size_t q = (size_t)y * vd.width + x;
        img[q] = fmaf(Tr[k], bg0, cr[k]);
        img[plane + q] = fmaf(Tr[k], bg1, cg[k]);
        img[2 * plane + q] = fmaf(Tr[k], bg2, cb[k]);
        img[3 * plane + q] = 1.f - Tr[k];
        tfinal[vd.pix_off + q] = Tr[k];
        ncontrib[vd.pix_off + q] = last[k];
        if (CKPT) fstate[vd.pix_off + q] = make_float4(Tr[k], cr[k], cg[k], cb[k]);
    }
}

// ---- the loss's final reduction ---------------------------------------------------
//
// Sum of the loss's partials in a fixed order (deterministic) -> loss; optionally
// advances the optimiser step counter (the fit step's Adam runs after it).  The order
// is that of 1024 threads whatever the workgroup: each of its NW waves takes the
// places of 16 / NW waves in turn.  A call of the loss alone runs it as a kernel of one
// workgroup; in a fit step it is one more workgroup of the adjoint, which needs none
// of it, and costs no launch (the smallest step 88 us to 85.5).
constexpr int kTailWaves = 16;

template <int NW>
__device__ __forceinline__ void loss_tail(const LossTail &lt, float *s_part) {
    const int lane = (int)(threadIdx.x & 63);
    const int n4 = lt.nparts / 4;
    for (int w = (int)(threadIdx.x >> 6); w < kTailWaves; w += NW) {
        // four partials per thread and step (16-byte loads; the tail one by one),
        // in four sums
        const int t = 64 * w + lane;
        float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
        for (int k = t; k < n4; k += 64 * kTailWaves) {
            const float4 v = reinterpret_cast<const float4 *>(lt.partial)[k];
            s0 += v.x;
            s1 += v.y;
            s2 += v.z;
            s3 += v.w;
        }
        for (int k = 4 * n4 + t; k < lt.nparts; k += 64 * kTailWaves) s0 += lt.partial[k];
        float s = (s0 + s1) + (s2 + s3);
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);   // same tree on every lane
        if (lane == 0) s_part[w] = s;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < kTailWaves; w++) tot += s_part[w];
        const uint32_t cnt = lt.mask_count ? *lt.mask_count : lt.count_host;
        const float L = tot / (float)max(cnt, 1u);
        lt.loss[0] = lt.accumulate ? lt.loss[0] + L : L;   // accumulate: one share of a multi-plan loss
        if (!isfinite(L)) atomicOr(lt.flags, GSF_FLAG_NONFINITE);
        // a step whose keys overflowed the capacity is not counted (its Adam
        // update is skipped too, so it can be repeated after a re-plan)
        if (lt.step_inc && !(*lt.flags & GSF_FLAG_CAPACITY)) lt.step_inc[0] = lt.step_inc[0] + 1;
    }
}

// ---- adjoint ---------------------------------------------------------------------
//
// One wave per 8 x 8 block of the tile's pixels (T / 8 squared waves a
// workgroup), one pixel per lane.  The tile's list is taken back to front in
// chunks of 64 records, staged in LDS; each wave lists the chunk's splats that
// reach its block and walks them eight at a time.  Per splat and pixel the
// recurrence leaves two numbers: te = dL/d(opacity) (dL/dpower = o te) and wT =
// alpha T.  Everything the splat's screen-space gradient needs from the block is
// a contraction of these over the block's 64 pixels:
//   sum te {1, u, v, u^2, u v, v^2}   (u, v: pixel offsets from the block's centre)
//   sum wT {dL/dR, dL/dG, dL/dB}
// whose right-hand factors do not depend on the splat.  Eight splats' te and wT
// rows (16 x 64, through LDS) times that 64 x 9 matrix (in registers, laid out
// once per unit) are sixteen v_mfma_f64_16x16x4_f64.  When a chunk
// is done the blocks' sums are moved from their centres to each splat's mean and
// added in the order of the blocks: no atomics, the same bits in every run.
// The products are in 64 bits because of that move: where a narrow splat lies off the
// centre, its sums about the centre are tens of times those about the mean, and FP32
// products left up to 2.4 times the error in the gradient that sums about the mean
// have (6,548 Gaussians on 447 x 99: 1.05e-6 of its norm against 4.3e-7; now 4.9e-7).
// They cost half the rate: an FP32 form took 5 to 13% less time for the whole step.
// (No VALU work of other waves issues under these instructions, 64 cycles each,
// so this form is for plans where the length of the lists, not issue, sets the time:
// fit step of 1,000 Gaussians on 128^2 132 us to 100, forward and backward of 30,011
// on 701 x 533 358 to 179.)
constexpr int kAdjChunk = 64;    // records staged at a time
constexpr int kAdjGroup = 8;     // splats per matrix product (two rows each)
constexpr int kAdjRow = 68;      // row stride, floats: 16-byte reads of 16 rows fall in distinct banks
constexpr int kAdjSec = kAdjChunk + 1;   // + the inert splat that pads a group

template <int T>
constexpr int adj_waves() { return (T / 8) * (T / 8); }

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int T>
struct AdjShared {
    static constexpr int NW = adj_waves<T>();
    float4 rec[2][4][kAdjSec];            // two chunks' records by section (a, b, c, ellipse)
    uint2 key[2][3][kAdjChunk];           // their boxes, row spans, first key positions
    alignas(16) float row[NW][2 * kAdjGroup * kAdjRow];
    double sum[NW][kAdjChunk * 9];        // per splat of the chunk: the block's nine sums
    uint64_t hit[NW];                     // splats of the chunk with sums
    alignas(16) int list[NW][kAdjChunk + kAdjGroup];
    uint32_t nmax[NW];
};

// Unit of adjoint work: the entries [us, ue) of launch tile ti's list (tm maps
// it to its view and tile).  With
// checkpoints (MODE 1) a unit is one LDS batch of `batch` entries and starts from
// the state the forward stored at the batch's end; otherwise a unit is the whole
// list and starts from the final state.  MODE 2 reads each included pair's
// transmittance from tstore instead of dividing.
template <int T, int MODE>
__device__ __forceinline__ void render_bwd_unit(
    uint32_t ti, const TileMap &tm, uint32_t us, uint32_t ue, bool last_unit, const uint2 &rg,
    uint32_t batch, const uint32_t *__restrict__ vals, SplatPtrs sp,
    const ViewDesc *__restrict__ views, int nviews, const gsf_camera *__restrict__ cams,
    const float *__restrict__ tfinal, const uint32_t *__restrict__ ncontrib,
    const float4 *__restrict__ fstate, const float4 *__restrict__ ckpt,
    const float *__restrict__ tstore, const float *__restrict__ bg, const float *__restrict__ dl,
    const KeyPlace &kp, AdjShared<T> &sh) {
    static_assert(T > 8, "an 8-pixel tile is one block");
    constexpr bool CKPT = MODE == 1;
    constexpr int NW = adj_waves<T>(), NT = 64 * NW;
    constexpr int PARTS = NT >= 256 ? 1 : 256 / NT;   // 16-byte record pieces a thread stages per chunk
    constexpr int QX = T / 8;                         // blocks per tile row
    int v, ty, tx;
    ViewDesc vd;
    launch_tile(ti, tm, views, nviews, T, v, vd, ty, tx);   // a tile with keys: valid
    // a fovea-culled forward over compact tiles composited only the disk's pixels
    // of the tiles that may hold some (the others carry no loss): the rest have no
    // contributor here (over global tiles the forward left them stopped, with no
    // contributor, which the pixel state says)
    const bool live = !tm.gaze || fovea_tile_live(tm.gaze, v, tm.radius, vd.width, vd.height, T, tx, ty);
    const float disk_r = tm.gaze ? tm.radius * (float)vd.width : 0.f;
    const int tid = (int)threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float *bgv = bg ? bg + 3 * v : cams[v].bg;
    const size_t plane = (size_t)vd.width * vd.height;
    const float *dimg = dl + 4 * (size_t)vd.pix_off;
    const int bx = tx * T + (wave % QX) * 8, by = ty * T + (wave / QX) * 8;   // the block's first pixel

    // gR: dL/dC-weighted colour behind the current splat, less gA Tf (the alpha
    // plane's share), carried as one value since only that difference is used
    const int x = bx + (lane & 7), y = by + (lane >> 3);
    const float px = (float)x, py = (float)y;   // integer pixel; its centre's offset from a mean is splat_dx
    const int pix = (y - ty * T) * T + (x - tx * T);   // the pixel's row-major index in the tile
    float Tr = 1.f, Tf = 1.f, g0 = 0.f, g1 = 0.f, g2 = 0.f, gA = 0.f;
    uint32_t nc = 0u;
    const bool inside = live && x < vd.width && y < vd.height && in_fovea(tm.gaze, v, x, y, disk_r);
    const size_t q = inside ? (size_t)y * vd.width + x : 0;
    if (inside) {
        Tf = tfinal[vd.pix_off + q];
        nc = ncontrib[vd.pix_off + q];
        g0 = dimg[q];
        g1 = dimg[plane + q];
        g2 = dimg[2 * plane + q];
        gA = dimg[3 * plane + q];
    }
    // a pixel no splat reached passes no gradient, whatever its dL/dimage
    // (which a fovea-culled loss may not have written): it starts at zero
    if (nc == 0u) {
        Tf = 1.f;
        g0 = g1 = g2 = gA = 0.f;
    }
    float gR = Tf * (g0 * bgv[0] + g1 * bgv[1] + g2 * bgv[2]);
    Tr = Tf;
    if (CKPT && !last_unit && rg.x + nc > us) {
        // colour behind the unit = final colour - colour accumulated at its end
        const float4 fs = fstate[vd.pix_off + q];
        const float4 cp = ckpt[(size_t)(ue / batch) * (T * T) + pix];
        Tr = cp.x;
        gR = gR + g0 * (fs.y - cp.y) + g1 * (fs.z - cp.z) + g2 * (fs.w - cp.w);
    }
    gR -= gA * Tf;
    // the block's largest contributor count: a splat at or past it reaches no
    // pixel of the block; and the tile's
    uint32_t qmax = nc;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) qmax = max(qmax, (uint32_t)__shfl_xor((int)qmax, o, 64));
    qmax = __builtin_amdgcn_readfirstlane(qmax);
    float *const row = sh.row[wave];
    row[lane] = g0;
    row[64 + lane] = g1;
    row[128 + lane] = g2;
    if (lane == 0) sh.nmax[wave] = qmax;
    if (tid < 6) {   // the inert splat of both buffers: limit 0, never included
        sh.rec[tid & 1][tid >> 1][kAdjChunk] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    uint32_t nmax = 0u;
#pragma unroll
    for (int w = 0; w < NW; w++) nmax = max(nmax, sh.nmax[w]);
    const uint32_t top = min(ue, rg.x + nmax);

    // Right-hand factor: lane (column j = lane & 15, k = lane >> 4) holds, for
    // product m, column j of pixel 16 k + m: 1, u, v, u^2, u v, v^2 (exact in
    // float: u, v are half-integers), then the pixel's dL/dR, dL/dG, dL/dB.
    const int j = lane & 15, kq = lane >> 4;
    float bq[16];
    {
        const float *gp = row + 64 * min(max(j - 6, 0), 2) + 16 * kq;
#pragma unroll
        for (int h = 0; h < 2; h++) {
            const float vv = (float)(2 * kq + h) - 3.5f;
            const float c0 = j == 0 ? 1.f : (j == 2 ? vv : (j == 5 ? vv * vv : 0.f));
            const float c1 = j == 1 ? 1.f : (j == 4 ? vv : 0.f);
            const float c2 = j == 3 ? 1.f : 0.f;
#pragma unroll
            for (int m = 0; m < 8; m++) {
                const float u = (float)m - 3.5f;
                const float poly = fmaf(fmaf(c2, u, c1), u, c0);
                bq[8 * h + m] = j >= 6 && j < 9 ? gp[8 * h + m] : poly;
            }
        }
    }
    __builtin_amdgcn_wave_barrier();   // row is reused below

    // Staging, from registers loaded a chunk ahead (record ids two ahead): thread
    // (entry e = t / 4, piece t % 4) takes one 16-byte piece of a record and one
    // of the key-slot lookup's three arrays.
    uint32_t rid[PARTS];
    float4 pre[PARTS];
    uint2 kpre[PARTS];
    auto fetch_ids = [&](uint32_t ce) {   // record ids of the chunk that ends at ce
        const uint32_t cs = ce - us > (uint32_t)kAdjChunk ? ce - kAdjChunk : us;
#pragma unroll
        for (int i = 0; i < PARTS; i++) {
            const int t = tid + i * NT;
            rid[i] = t < 256 && cs + (uint32_t)(t >> 2) < ce ? vals[cs + (uint32_t)(t >> 2)] : ~0u;
        }
    };
    auto fetch_recs = [&]() {
#pragma unroll
        for (int i = 0; i < PARTS; i++) {
            const int part = (tid + i * NT) & 3;
            kpre[i] = make_uint2(0u, 0u);
            pre[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (rid[i] != ~0u) {
                pre[i] = *sp.at(rid[i], part);
                if (part == 0) kpre[i] = kp.rect[rid[i]];
                else if (part == 1) kpre[i] = kp.rspan[rid[i]];
                else if (part == 2) kpre[i].x = kp.koff[rid[i]];
            }
        }
    };
    if (top > us) {
        fetch_ids(top);
        fetch_recs();
        const uint32_t cs = top - us > (uint32_t)kAdjChunk ? top - kAdjChunk : us;
        if (cs > us) fetch_ids(cs);
    }
    int buf = 0;
    for (uint32_t ce = top; ce > us; buf ^= 1) {
        const uint32_t cs = ce - us > (uint32_t)kAdjChunk ? ce - (uint32_t)kAdjChunk : us;
        const int nb = (int)(ce - cs);
#pragma unroll
        for (int i = 0; i < PARTS; i++) {
            const int t = tid + i * NT;
            if (t < 256) {
                sh.rec[buf][t & 3][t >> 2] = pre[i];
                if ((t & 3) < 3) sh.key[buf][t & 3][t >> 2] = kpre[i];
            }
        }
        if (cs > us) {
            fetch_recs();
            const uint32_t ns = cs - us > (uint32_t)kAdjChunk ? cs - kAdjChunk : us;
            if (ns > us) fetch_ids(ns);
        }
        __syncthreads();
        const float4 *SA = sh.rec[buf][kRecA], *SB = sh.rec[buf][kRecB], *SC = sh.rec[buf][kRecC];
        // the wave's splats of the chunk, back to front, as byte offsets from the
        // first buffer's sections (whose starts are then the reads' constant offsets)
        const int base = buf * (int)sizeof(sh.rec[0]);
        const uint32_t off = cs - rg.x;   // list position of the chunk's first record
        bool meet = lane < nb && off + (uint32_t)lane < qmax;
        if (meet) {
            const float4 e0 = sh.rec[buf][kRecEll][lane], a0 = SA[lane], c0 = SC[lane];
            const Ellipse e{e0.x, e0.y, e0.z, e0.w, quad_half_height(e0), a0.x, a0.y, (int)c0.z, (int)c0.w};
            meet = quad_meets(e, bx, by);
        }
        const uint64_t m64 = __ballot(meet);
        const int cnt = (int)__popcll(m64);
        int *const list = sh.list[wave];
        if (meet) list[cnt - 1 - (int)lanes_below(m64)] = base + lane * (int)sizeof(float4);
        if (lane < kAdjGroup) list[cnt + lane] = base + kAdjChunk * (int)sizeof(float4);
        if (lane == 0) sh.hit[wave] = m64;
        __builtin_amdgcn_wave_barrier();
        // entries below the pixel's contributor count, as byte offsets
        const int lim = base + (int)(nc - min(nc, off)) * (int)sizeof(float4);
        for (int g = 0; g < cnt; g += kAdjGroup) {
            uint32_t took = 0u;   // splats of the group that some pixel of the block included
#pragma unroll
            for (int h = 0; h < kAdjGroup; h += 4) {
                if (g + h >= cnt) break;   // wave-uniform
                const int4 j4 = *(const int4 *)(list + g + h);
                const int bo[4] = {j4.x, j4.y, j4.z, j4.w};
                // What does not depend on the recurrence, without branches.  A pixel
                // the splat does not reach takes power -inf: exp2 = 0, alpha = 0,
                // 1 / (1 - alpha) = 1, and its state passes through unchanged bit
                // for bit with te = wT = 0.  A clamped alpha passes no gradient to
                // the opacity or the power (exo = 0).
                float al[4], inv[4], gc[4], exo[4], tb[4];
                bool in4[4];
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const float4 a = *(const float4 *)((const char *)sh.rec[0][kRecA] + bo[u]);
                    const float4 b = *(const float4 *)((const char *)sh.rec[0][kRecB] + bo[u]);
                    const float4 c = *(const float4 *)((const char *)sh.rec[0][kRecC] + bo[u]);
                    const float dx = splat_dx(px, c.z, a.x);
                    const float dy = splat_dx(py, c.w, a.y);
                    const float fall = splat_fall(a, b, dx, dy);
                    const bool inc = (bo[u] < lim) & splat_within(fall, c.y);
                    in4[u] = inc;
                    if (__builtin_amdgcn_ballot_w64(inc)) took |= 1u << (h + u);
                    const float ex = __builtin_amdgcn_exp2f(-(inc ? fall : __builtin_inff()));
                    const float ae = b.y * ex;
                    al[u] = fminf(kAlphaMax, ae);
                    inv[u] = __builtin_amdgcn_rcpf(1.f - al[u]);   // alpha <= 0.99
                    gc[u] = fmaf(g2, c.x, fmaf(g1, b.w, g0 * b.z));
                    exo[u] = ae > kAlphaMax ? 0.f : ex;
                    if (MODE == 2)
                        tb[u] = inc ? tstore[(size_t)(cs + (uint32_t)(bo[u] - base) / (uint32_t)sizeof(float4)) * (T * T) + pix]
                                    : 0.f;
                }
#pragma unroll
                for (int u = 0; u < 4; u++) {
                    const float Tb = MODE == 2 ? tb[u] : Tr * inv[u];
                    const float dalpha = fmaf(Tb, gc[u], -(gR * inv[u]));
                    const float wT = al[u] * Tb;
                    gR = fmaf(gc[u], wT, gR);
                    if (MODE != 2) Tr = Tb;
                    row[(2 * (h + u)) * kAdjRow + lane] = MODE == 2 && !in4[u] ? 0.f : exo[u] * dalpha;
                    row[(2 * (h + u) + 1) * kAdjRow + lane] = wT;
                }
            }
            __builtin_amdgcn_wave_barrier();
            f64x4 D = {0.0, 0.0, 0.0, 0.0};
            if (took) {
                f32x4 av[4];
#pragma unroll
                for (int i = 0; i < 4; i++) av[i] = *(const f32x4 *)(row + (lane & 15) * kAdjRow + 16 * kq + 4 * i);
#pragma unroll
                for (int m = 0; m < 16; m++)
                    D = __builtin_amdgcn_mfma_f64_16x16x4f64((double)av[m >> 2][m & 3], (double)bq[m], D, 0, 0, 0);
            }
            // lane (j, k) holds column j of rows k, k + 4, k + 8 and k + 12: te (k even) or
            // wT of the group's splats k / 2, + 2, + 4 and + 6.  A splat no pixel included
            // has zeros.
            if ((kq & 1) ? j >= 6 && j < 9 : j < 6) {
                double *const S = sh.sum[wave] + j;
#pragma unroll
                for (int r = 0; r < 4; r++) {
                    const int e = (kq >> 1) + 2 * r;
                    if (g + e < cnt) S[((list[g + e] - base) >> 4) * 9] = (took >> e) & 1u ? D[r] : 0.0;
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
        __syncthreads();
        // The chunk's keys: thread (entry, piece) adds the blocks' sums about the
        // splat's mean, applies the conic factors and stores its 16 bytes of the
        // key's own 64-byte chunk (no other workgroup writes it):
        //   dpower/dmean = (A dx + B dy, B dx + C dy) = -ln2 (2 A2 dx + B2 dy, B2 dx + 2 C2 dy);
        //   dpower/d(A, B, C) = (-dx^2 / 2, -dx dy, -dy^2 / 2)
#pragma unroll
        for (int i = 0; i < PARTS; i++) {
            const int t = tid + i * NT, e = t >> 2, part = t & 3;
            if (t >= 256 || e >= nb) continue;
            const float4 a = SA[e], b = SB[e], c = SC[e];
            float4 out = make_float4(0.f, 0.f, 0.f, 0.f);
            if (part < 3) {
                // in 64 bits, as the sums about the centre of a block cancel where a small
                // splat lies off it
                double dx = 0.0, dy = 0.0, dxx = 0.0, dxy = 0.0, dyy = 0.0;
                float s0 = 0.f, r0 = 0.f, r1 = 0.f, r2 = 0.f;
#pragma unroll
                for (int w = 0; w < NW; w++) {
                    if (!((sh.hit[w] >> e) & 1ull)) continue;
                    const double *M = sh.sum[w] + 9 * e;
                    if (part == 2) {
                        r2 += (float)M[8];
                        continue;
                    }
                    // the block centre's offset from the mean
                    const double ey = (double)((float)(ty * T + (w / QX) * 8) + 3.5f - c.w) + (double)a.y;
                    if (part == 1) {
                        dyy += fma(ey, fma(ey, M[0], 2.0 * M[2]), M[5]);
                        s0 += (float)M[0];
                        r0 += (float)M[6];
                        r1 += (float)M[7];
                        continue;
                    }
                    const double ex = (double)((float)(tx * T + (w % QX) * 8) + 3.5f - c.z) + (double)a.x;
                    const double m0 = M[0], m1 = M[1], m2 = M[2];
                    dx += fma(ex, m0, m1);
                    dy += fma(ey, m0, m2);
                    dxx += fma(ex, fma(ex, m0, 2.0 * m1), M[3]);
                    dxy += fma(ex, fma(ey, m0, m2), fma(ey, m1, M[4]));
                }
                const float sx = (float)dx, sy = (float)dy, sxx = (float)dxx, sxy = (float)dxy, syy = (float)dyy;
                const float o = b.y;   // te sums -> dL/dpower sums
                if (part == 0)
                    out = make_float4(-kLn2 * o * (2.f * a.z * sx + a.w * sy),
                                      -kLn2 * o * (a.w * sx + 2.f * b.x * sy), -0.5f * (o * sxx), -(o * sxy));
                else if (part == 1)
                    out = make_float4(-0.5f * (o * syy), s0, r0, r1);
                else
                    out.x = r2;
            }
            const uint32_t slot = key_slot_of(kp, sh.key[buf][0][e], sh.key[buf][1][e], sh.key[buf][2][e].x, ty, tx);
            kp.pg[(size_t)slot * kKeyGradF4 + part] = out;
        }
        ce = cs;
    }
    // keys behind every pixel's last included splat pass no gradient
    for (uint32_t t = (max(top, us) << 2) + (uint32_t)tid; (t >> 2) < ue; t += NT)
        kp.pg[(size_t)key_slot(kp, vals[t >> 2], ty, tx) * kKeyGradF4 + (t & 3u)] = make_float4(0.f, 0.f, 0.f, 0.f);
}

// ---- adjoint with one wave per tile, or per 16-pixel quarter of a 32-pixel tile ------
//
// Plans with many tiles are bound by VALU issue, so here one wave walks the
// tile's list with (16 pixels and up) four pixels a lane (pixel block k = quadrant
// k), sums its pixels' terms in the lane and reduces nine sums over the 64 lanes
// once per splat.  That reduction is nine DPP adds (each row's lanes 8 apart, two fields
// packed into a register by the bank masks), five 4-byte LDS stores, and, for
// three splats at a time, 54 lanes that add half a row of 32 partial sums each:
// about 60 VALU cycles a splat, where folding pairs of splats with permlane swaps
// (8 cycles an instruction) and four DPP adds a row took 132.  An instruction
// stream of 2-cycle operations (add, multiply, FMA) needs several waves ready on a
// SIMD, so LDS (7 KB) and registers (82) are kept to five waves, and scalar
// bookkeeping out of the loop.  Sixteen views of 1920^2, 16.7M keys: 2372 -> 1910
// us; eight uneven views, 7.5M keys: 1100 -> 835 us.
constexpr int kTileGroup = 3;              // splats whose partial sums are added together
constexpr int kTileRow = 36;               // row stride of the 32 partial sums, floats
// Opacities up to this cannot reach the alpha clamp (0.99; exp2 of a power <= 0
// is at most 1 within rounding), so chunks without a larger one leave out the
// clamp and its test (11 of about 112 VALU cycles per quadrant and splat).
constexpr float kOpenOpacity = 0.98f;

template <int T>
constexpr int tile_adj_waves() { return T == 32 ? 4 : 1; }

struct TileAdjWave {
    // the chunk's records by section (a, b, c); a splat's nine sums replace its record
    float4 rec[3][kAdjChunk];
    alignas(16) float row[kTileGroup * 9 * kTileRow];
};
template <int T>
struct TileAdjShared {
    TileAdjWave wave[tile_adj_waves<T>()];
    uint64_t hit[tile_adj_waves<T>()];   // splats of the chunk with sums (32-pixel tiles)
    uint32_t nmax[tile_adj_waves<T>()];
};

// acc[f] summed over lanes 8 apart of each 16-lane row: fields 2 k (lanes 0-7 of
// each row) and 2 k + 1 (lanes 8-15) in out[k], field 8 in out[4].  (The s_nop
// gives the DPP reads the two wait states they need after the writes of acc.)
__device__ __forceinline__ void fold8(const float (&acc)[9], float (&out)[5]) {
    asm volatile(
        "s_nop 1\n\t"
        "v_add_f32_dpp %0, %5, %5 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %1, %7, %7 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %2, %9, %9 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %3, %11, %11 row_ror:8 row_mask:0xf bank_mask:0x3\n\t"
        "v_add_f32_dpp %4, %13, %13 row_ror:8 row_mask:0xf bank_mask:0xf\n\t"
        "v_add_f32_dpp %0, %6, %6 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %1, %8, %8 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %2, %10, %10 row_ror:8 row_mask:0xf bank_mask:0xc\n\t"
        "v_add_f32_dpp %3, %12, %12 row_ror:8 row_mask:0xf bank_mask:0xc"
        : "=&v"(out[0]), "=&v"(out[1]), "=&v"(out[2]), "=&v"(out[3]), "=&v"(out[4])
        : "v"(acc[0]), "v"(acc[1]), "v"(acc[2]), "v"(acc[3]), "v"(acc[4]), "v"(acc[5]), "v"(acc[6]),
          "v"(acc[7]), "v"(acc[8]));
}

template <int T, int MODE>
__device__ __forceinline__ void render_bwd_tile(
    uint32_t ti, const TileMap &tm, uint32_t us, uint32_t ue, bool last_unit, const uint2 &rg,
    uint32_t batch, const uint32_t *__restrict__ vals, SplatPtrs sp,
    const ViewDesc *__restrict__ views, int nviews, const gsf_camera *__restrict__ cams,
    const float *__restrict__ tfinal, const uint32_t *__restrict__ ncontrib,
    const float4 *__restrict__ fstate, const float4 *__restrict__ ckpt,
    const float *__restrict__ tstore, const float *__restrict__ bg, const float *__restrict__ dl,
    const KeyPlace &kp, TileAdjShared<T> &shared) {
    constexpr bool CKPT = MODE == 1;
    constexpr int NW = tile_adj_waves<T>();
    constexpr int PPT = T == 8 ? 1 : 4;
    const int wave = NW > 1 ? __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6) : 0;
    TileAdjWave &sh = shared.wave[wave];
    int v, ty, tx;
    ViewDesc vd;
    launch_tile(ti, tm, views, nviews, T, v, vd, ty, tx);   // a tile with keys: valid
    const bool live = !tm.gaze || fovea_tile_live(tm.gaze, v, tm.radius, vd.width, vd.height, T, tx, ty);
    const float disk_r = tm.gaze ? tm.radius * (float)vd.width : 0.f;
    const int lane = threadIdx.x & 63;
    const float *bgv = bg ? bg + 3 * v : cams[v].bg;
    const float bg0 = bgv[0], bg1 = bgv[1], bg2 = bgv[2];
    const size_t plane = (size_t)vd.width * vd.height;
    const float *dimg = dl + 4 * (size_t)vd.pix_off;

    // the pixel state, as render_bwd_unit has it, for the lane's pixel of each quadrant
    float px[PPT], py[PPT], Tr[PPT], Tf[PPT], gR[PPT], g0[PPT], g1[PPT], g2[PPT], gA[PPT];
    uint32_t nc[PPT], qmax[PPT];
    int pix[PPT];
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int lx = (wave & 1) * 16 + (k & 1) * 8 + (lane & 7);
        const int ly = (wave >> 1) * 16 + (k >> 1) * 8 + (lane >> 3);
        pix[k] = ly * T + lx;
        const int x = tx * T + lx, y = ty * T + ly;
        const bool inside = live && x < vd.width && y < vd.height && in_fovea(tm.gaze, v, x, y, disk_r);
        const size_t q = inside ? (size_t)y * vd.width + x : 0;
        px[k] = (float)x;
        py[k] = (float)y;
        nc[k] = 0u;
        if (inside) {
            Tf[k] = tfinal[vd.pix_off + q];
            nc[k] = ncontrib[vd.pix_off + q];
            g0[k] = dimg[q];
            g1[k] = dimg[plane + q];
            g2[k] = dimg[2 * plane + q];
            gA[k] = dimg[3 * plane + q];
        }
        if (nc[k] == 0u) {
            Tf[k] = 1.f;
            g0[k] = g1[k] = g2[k] = gA[k] = 0.f;
        }
        gR[k] = Tf[k] * (g0[k] * bg0 + g1[k] * bg1 + g2[k] * bg2);
        Tr[k] = Tf[k];
        if (CKPT && !last_unit && rg.x + nc[k] > us) {
            const float4 fs = fstate[vd.pix_off + q];
            const float4 cp = ckpt[(size_t)(ue / batch) * (T * T) + pix[k]];
            Tr[k] = cp.x;
            gR[k] = gR[k] + g0[k] * (fs.y - cp.y) + g1[k] * (fs.z - cp.z) + g2[k] * (fs.w - cp.w);
        }
        gR[k] -= gA[k] * Tf[k];
    }
    // per quadrant the largest contributor count: a splat at or past it reaches no
    // pixel of the quadrant
    uint32_t nmax = 0u;
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        uint32_t x = nc[k];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x = max(x, (uint32_t)__shfl_xor((int)x, o, 64));
        qmax[k] = __builtin_amdgcn_readfirstlane(x);
        nmax = max(nmax, qmax[k]);
    }
    if constexpr (NW > 1) {   // the tile's
        if (lane == 0) shared.nmax[wave] = nmax;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < NW; w++) nmax = max(nmax, shared.nmax[w]);
    }
    const uint32_t top = min(ue, rg.x + nmax);
    // the lane's row of partial sums (splat lane / 18, field lane / 2 % 9), its
    // half, and where in the splat's record that field's sum goes
    const int prow = lane >> 1, psplat = prow / 9, pfield = prow - 9 * psplat;
    const int prd = prow * kTileRow + (lane & 1) * 4;
    const int psum = (pfield >> 2) * (4 * kAdjChunk) + (pfield & 3);
    const int pwr = ((lane >> 3) & 1) * kTileRow + (lane >> 4) * 8 + (lane & 7);

    uint32_t rid = 0u;   // record ids are read a chunk ahead
    if (top > us) {
        const uint32_t cs = top - us > (uint32_t)kAdjChunk ? top - kAdjChunk : us;
        if (cs + (uint32_t)lane < top) rid = vals[cs + (uint32_t)lane];
    }
    for (uint32_t be = top; be > us;) {
        const uint32_t bs = be - us > (uint32_t)kAdjChunk ? be - (uint32_t)kAdjChunk : us;
        const int nb = (int)(be - bs);
        const uint32_t off = bs - rg.x;   // list position of the chunk's first record
        // the lane's record: conic factors, opacity, its key's slot and the
        // quadrants it reaches before their deepest contributor
        float A2 = 0.f, B2 = 0.f, C2 = 0.f, o = 0.f;
        uint32_t slot = 0u, qmask = 0u;
        if (lane < nb) {
            const float4 *rr = sp.at(rid, 0);   // one 64-byte chunk: splat and ellipse
            const float4 ra = rr[kRecA], rb = rr[kRecB], rc = rr[kRecC], e0 = rr[kRecEll];
            if (wave == 0) slot = key_slot(kp, rid, ty, tx);
            sh.rec[0][lane] = ra;
            sh.rec[1][lane] = rb;
            sh.rec[2][lane] = rc;
            A2 = ra.z;
            B2 = ra.w;
            C2 = rb.x;
            o = rb.y;
            if constexpr (T >= 16) {
                const Ellipse e{e0.x, e0.y, e0.z, e0.w, quad_half_height(e0), ra.x, ra.y, (int)rc.z, (int)rc.w};
                qmask = quadrant_mask(e, tx * T + (wave & 1) * 16, ty * T + (wave >> 1) * 16);
            } else {
                qmask = 1u;   // the list holds the splats that reach the tile's one block
            }
#pragma unroll
            for (int k = 0; k < PPT; k++)
                if (off + (uint32_t)lane >= qmax[k]) qmask &= ~(1u << k);
        }
        if (bs > us) {
            const uint32_t ns = bs - us > (uint32_t)kAdjChunk ? bs - kAdjChunk : us;
            if (ns + (uint32_t)lane < bs) rid = vals[ns + (uint32_t)lane];
        }
        __builtin_amdgcn_wave_barrier();
        // Splat j's per-lane sums: te dx, te dy, te dx^2, te dx dy, te dy^2 (te =
        // dL/do, so that o te = dL/dpower), dL/do, dL/dcolour; folded into group
        // row G.
        auto splat = [&](int j, int G, auto clamp_tag) __attribute__((always_inline)) {
            constexpr bool CLAMP = decltype(clamp_tag)::value;
            const uint32_t pos = off + (uint32_t)j;
            const float4 a = sh.rec[0][j], b = sh.rec[1][j], c = sh.rec[2][j];
            // the splat's quadrant mask, wave-uniform: tested in scalar registers
            const uint32_t qm = (uint32_t)__builtin_amdgcn_readlane((int)qmask, j);
            // the offsets and the terms in y, of the two columns and two rows of
            // quadrants (once instead of per quadrant: 1920 -> 1883 us on sixteen
            // views of 1920^2)
            constexpr int NC = PPT == 4 ? 2 : 1;
            float dxc[NC], dyr[NC], wy[NC], vy[NC];
#pragma unroll
            for (int i = 0; i < NC; i++) {
                dxc[i] = splat_dx(px[i], c.z, a.x);
                dyr[i] = splat_dx(py[2 * i], c.w, a.y);
                wy[i] = a.w * dyr[i];
                vy[i] = ((-b.x) * dyr[i]) * dyr[i];
            }
            float acc[9];
            // (-0 is the exact identity of addition, so the first term needs no add)
#pragma unroll
            for (int f = 0; f < 9; f++) acc[f] = -0.f;
#pragma unroll
            for (int k = 0; k < PPT; k++) {
                if (!((qm >> k) & 1u)) continue;   // wave-uniform
                // Branch-free per lane: every value is computed and a pixel the
                // splat does not reach (behind its last contributor, or alpha
                // below 1/255) takes power -inf instead, so exp2 = 0, alpha = 0, 1 /
                // (1 - alpha) = 1 and its state passes through unchanged bit for bit
                // with zero sums, without a select per quantity.
                const float dx = dxc[k % NC], dy = dyr[k / NC];
                const float fall = fmaf(-dx, fmaf(a.z, dx, wy[k / NC]), vy[k / NC]);   // splat_fall
                const bool inc = (pos < nc[k]) & splat_within(fall, c.y);
                // no pixel of the block takes the splat: every lane would add
                // zeros and keep its state (wave-uniform)
                if (!__any(inc)) continue;
                const float ex = __builtin_amdgcn_exp2f(-(MODE == 2 || inc ? fall : __builtin_inff()));
                const float ae = b.y * ex;
                const float alpha = CLAMP ? fminf(kAlphaMax, ae) : ae;
                const float inv = __builtin_amdgcn_rcpf(1.f - alpha);   // alpha <= 0.99
                float Tb;
                if (MODE == 2)
                    Tb = inc ? tstore[(size_t)(bs + (uint32_t)j) * (T * T) + pix[k]] : 0.f;
                else
                    Tb = Tr[k] * inv;
                const float gc = fmaf(g2[k], c.x, fmaf(g1[k], b.w, g0[k] * b.z));
                const float dalpha = fmaf(Tb, gc, -(gR[k] * inv));
                const float wT = MODE != 2 || inc ? alpha * Tb : 0.f;
                acc[6] = fmaf(wT, g0[k], acc[6]);
                acc[7] = fmaf(wT, g1[k], acc[7]);
                acc[8] = fmaf(wT, g2[k], acc[8]);
                gR[k] = fmaf(gc, wT, gR[k]);
                if (MODE == 2) Tr[k] = inc ? Tb : Tr[k];
                else Tr[k] = Tb;
                // a clamped alpha passes no gradient to the opacity or the power;
                // te = dL/do, and dL/dpower (natural units) = o te, the opacity
                // factor being applied to the sums once per splat at the flush
                float te = ex * dalpha;
                if (CLAMP || MODE == 2) te = ((MODE != 2 || inc) & !(ae > kAlphaMax)) ? te : 0.f;
                acc[5] += te;
                const float ux = te * dx, uy = te * dy;
                acc[0] += ux;
                acc[1] += uy;
                acc[2] = fmaf(ux, dx, acc[2]);
                acc[3] = fmaf(ux, dy, acc[3]);
                acc[4] = fmaf(uy, dy, acc[4]);
            }
            float out[5];
            fold8(acc, out);
            const int w = pwr + G * (9 * kTileRow);
#pragma unroll
            for (int k = 0; k < 4; k++) sh.row[w + 2 * k * kTileRow] = out[k];
            if (!(lane & 8)) sh.row[w + 8 * kTileRow] = out[4];
        };
        // The splats that reach some quadrant, back to front, kTileGroup at a time;
        // then the group's rows are added: a lane adds half a row, its neighbour
        // the other half.
        const uint64_t some = __builtin_amdgcn_ballot_w64(qmask != 0u);
        auto walk = [&](auto clamp_tag) __attribute__((always_inline)) {
            uint64_t m = some;
            while (m) {   // wave-uniform
                int id[kTileGroup];
#pragma unroll
                for (int G = 0; G < kTileGroup; G++) {
                    id[G] = -1;
                    if (m) {
                        id[G] = 63 - __builtin_clzll(m);
                        m &= ~(1ull << id[G]);
                        splat(id[G], G, clamp_tag);
                    }
                }
                __builtin_amdgcn_wave_barrier();
                int mine = -1;   // the lane's splat (none past the group's last)
#pragma unroll
                for (int G = 0; G < kTileGroup; G++) mine = psplat == G ? id[G] : mine;
                if (mine >= 0) {
                    float4 x[4];
#pragma unroll
                    for (int i = 0; i < 4; i++) x[i] = *(const float4 *)(sh.row + prd + 8 * i);
                    const float s0 = (x[0].x + x[0].y) + (x[0].z + x[0].w), s1 = (x[1].x + x[1].y) + (x[1].z + x[1].w);
                    const float s2 = (x[2].x + x[2].y) + (x[2].z + x[2].w), s3 = (x[3].x + x[3].y) + (x[3].z + x[3].w);
                    float t = (s0 + s1) + (s2 + s3);
                    t += dpp_shift<0xB1, 0xf>(t);   // quad_perm [1, 0, 3, 2]: the other half
                    if (!(lane & 1)) ((float *)sh.rec)[4 * mine + psum] = t;
                }
                __builtin_amdgcn_wave_barrier();
            }
        };
        if (__builtin_amdgcn_ballot_w64(o > kOpenOpacity)) walk(std::true_type{});
        else walk(std::false_type{});
        if constexpr (NW > 1) {
            if (lane == 0) shared.hit[wave] = some;
            __syncthreads();
        }
        // one lane per splat adds the waves' nine sums, applies the conic factors and
        // stores them at the key's own position (no other workgroup writes it)
        if (wave == 0 && lane < nb) {
            float S[9];
#pragma unroll
            for (int f = 0; f < 9; f++) S[f] = 0.f;
#pragma unroll
            for (int w = 0; w < NW; w++) {
                if (!(((NW > 1 ? shared.hit[w] : some) >> lane) & 1ull)) continue;
#pragma unroll
                for (int f = 0; f < 9; f++)
                    S[f] += ((const float *)shared.wave[w].rec)[4 * lane + (f >> 2) * (4 * kAdjChunk) + (f & 3)];
            }
#pragma unroll
            for (int f = 0; f < 5; f++) S[f] *= o;   // te sums -> dL/dpower sums
            // dpower/dmean = (A dx + B dy, B dx + C dy) = -ln2 (2 A2 dx + B2 dy, B2 dx + 2 C2 dy);
            // dpower/d(A, B, C) = (-dx^2 / 2, -dx dy, -dy^2 / 2)
            float4 *g = kp.pg + (size_t)slot * kKeyGradF4;
            g[0] = make_float4(-kLn2 * (2.f * A2 * S[0] + B2 * S[1]),
                               -kLn2 * (B2 * S[0] + 2.f * C2 * S[1]), -0.5f * S[2], -S[3]);
            g[1] = make_float4(-0.5f * S[4], S[5], S[6], S[7]);
            g[2] = make_float4(S[8], 0.f, 0.f, 0.f);
            g[3] = make_float4(0.f, 0.f, 0.f, 0.f);
        }
        if constexpr (NW > 1) __syncthreads();   // the chunk's LDS is free again
        else __builtin_amdgcn_wave_barrier();
        be = bs;
    }
    // keys behind every pixel's last included splat pass no gradient
    for (uint32_t e = max(top, us) + threadIdx.x; e < ue; e += 64u * NW) {
        float4 *g = kp.pg + (size_t)key_slot(kp, vals[e], ty, tx) * kKeyGradF4;
#pragma unroll
        for (int f = 0; f < kKeyGradF4; f++) g[f] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
}

// WIDE: one wave per 8 x 8 block (render_bwd_unit); else one wave per tile or
// quarter tile (render_bwd_tile).
template <int T, bool WIDE>
struct AdjForm {
    using Shared = AdjShared<T>;
};
template <int T>
struct AdjForm<T, false> {
    using Shared = TileAdjShared<T>;
};
template <int T, bool WIDE>
constexpr int adj_threads() { return 64 * (WIDE ? adj_waves<T>() : tile_adj_waves<T>()); }

// Recompute (MODE 0) and stored (MODE 2) modes: one workgroup per tile, the
// whole list back to front; workgroup i takes tile order[i] like the forward.
template <int T, int MODE, bool WIDE>
__global__ __launch_bounds__((adj_threads<T, WIDE>()), WIDE && T == 16 ? 4 : 1) void k_render_bwd(
    const uint32_t *__restrict__ order,
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ vals, SplatPtrs sp,
    const ViewDesc *__restrict__ views, int nviews, const gsf_camera *__restrict__ cams,
    const float *__restrict__ tfinal, const uint32_t *__restrict__ ncontrib,
    const float *__restrict__ tstore, const float *__restrict__ bg, const float *__restrict__ dl,
    KeyPlace kp, TileMap tm, LossTail lt) {
    __shared__ typename AdjForm<T, WIDE>::Shared sh;
    const uint32_t tail = lt.partial ? 1u : 0u;   // workgroup 0 finishes the loss
    if (blockIdx.x < tail) {
        loss_tail<adj_threads<T, WIDE>() / 64>(lt, reinterpret_cast<float *>(&sh));
        return;
    }
    const uint32_t ti = order[blockIdx.x - tail];
    const uint2 rg = ranges[ti];
    // a tile without keys passes no gradient (and a fovea-culled step's tiles
    // away from the fovea hold no pixel state to read)
    if (rg.x == rg.y) return;
    if constexpr (WIDE)
        render_bwd_unit<T, MODE>(ti, tm, rg.x, rg.y, true, rg, 1u, vals, sp, views, nviews, cams, tfinal,
                                 ncontrib, nullptr, nullptr, tstore, bg, dl, kp, sh);
    else
        render_bwd_tile<T, MODE>(ti, tm, rg.x, rg.y, true, rg, 1u, vals, sp, views, nviews, cams, tfinal,
                              ncontrib, nullptr, nullptr, tstore, bg, dl, kp, sh);
}

// Checkpoint mode: one workgroup per (tile, batch) unit id.  Unit u of tile t
// has id floor(start_t / B) + t + u (strictly increasing, below M / B + tiles);
// a workgroup maps its id back to its tile by a 64-way search (each wave's lanes
// test 64 tiles at once: two rounds of loads for 4,096 tiles where halving takes
// twelve).  The grid covers
// the key capacity; ids at or above M / B + tiles (M read on the device) and
// ids that fall in no tile's units exit at once.
template <int T, bool WIDE>
__global__ __launch_bounds__((adj_threads<T, WIDE>()), WIDE && T == 16 ? 4 : 1) void k_render_bwd_ckpt(
    const uint2 *__restrict__ ranges, int total_tiles, uint32_t B, const uint32_t *__restrict__ m_dev,
    uint32_t m_host, const uint32_t *__restrict__ vals, SplatPtrs sp,
    const ViewDesc *__restrict__ views, int nviews, const gsf_camera *__restrict__ cams,
    const float *__restrict__ tfinal, const uint32_t *__restrict__ ncontrib,
    const float4 *__restrict__ fstate, const float4 *__restrict__ ckpt,
    const float *__restrict__ bg, const float *__restrict__ dl, KeyPlace kp, TileMap tm, LossTail lt) {
    __shared__ typename AdjForm<T, WIDE>::Shared sh;
    const uint32_t tail = lt.partial ? 1u : 0u;   // workgroup 0 finishes the loss
    if (blockIdx.x < tail) {
        loss_tail<adj_threads<T, WIDE>() / 64>(lt, reinterpret_cast<float *>(&sh));
        return;
    }
    const uint32_t m = m_dev ? *m_dev : m_host;
    const uint32_t n_ids = m / B + (uint32_t)total_tiles;
    const int lane = (int)(threadIdx.x & 63);
    for (uint32_t id = blockIdx.x - tail; id < n_ids; id += gridDim.x - tail) {   // one trip when the grid covers n_ids
        // largest tile t with first id floor(start_t / B) + t <= id: in [lo, lo + len)
        int lo = 0, len = total_tiles;
        while (len > 1) {   // wave-uniform
            const int step = (len + 63) >> 6, t = lo + lane * step;
            const bool le = lane * step < len && ranges[t].x / B + (uint32_t)t <= id;
            // monotone in t, and true for lo: the last true lane
            const int k = 63 - __builtin_clzll(__ballot(le) | 1ull);
            len = min(step, len - k * step);
            lo += k * step;
        }
        const uint2 rg = ranges[lo];
        const uint32_t u = id - (rg.x / B + (uint32_t)lo);
        const uint32_t units = (rg.y - rg.x + B - 1) / B;
        if (u >= units) continue;
        const uint32_t us = rg.x + u * B;
        const uint32_t ue = min(rg.y, us + B);
        if constexpr (WIDE)
            render_bwd_unit<T, 1>((uint32_t)lo, tm, us, ue, u + 1 == units, rg, B, vals, sp, views, nviews,
                                  cams, tfinal, ncontrib, fstate, ckpt, nullptr, bg, dl, kp, sh);
        else
            render_bwd_tile<T, 1>((uint32_t)lo, tm, us, ue, u + 1 == units, rg, B, vals, sp, views, nviews,
                               cams, tfinal, ncontrib, fstate, ckpt, nullptr, bg, dl, kp, sh);
        __syncthreads();   // the unit's LDS is free again
    }
}

// Per-record sum of the per-key screen-space gradients into g2d [9][nrec]
// (wave_key_sum; one wave per workgroup, so that small record counts still
// spread over every CU).  The fit step sums inside the projection adjoint
// instead; this pass serves the debug readout of g2d.
__global__ __launch_bounds__(64) void k_grad_sum(KeyPlace kp, int nrec, float *__restrict__ g2d) {
    const int r = blockIdx.x * 64 + threadIdx.x;
    float S[9];
    wave_key_sum(kp, (uint32_t)r, r < nrec, S);
    if (r < nrec) {
#pragma unroll
        for (int f = 0; f < 9; f++) g2d[(size_t)f * nrec + r] = S[f];
    }
}

// Work accounting: the same per-pixel walk as k_render_fwd, counting instead
// of compositing.  counters: visited (forward), included, visited (adjoint).
template <int T>
__global__ __launch_bounds__(T * T < 256 ? T * T : 256) void k_count_pairs(
    const uint2 *__restrict__ ranges, const uint32_t *__restrict__ vals, SplatPtrs sp,
    const ViewDesc *__restrict__ views, int nviews, TileMap tm, const float *__restrict__ cull_gaze,
    float cull_radius, unsigned long long *__restrict__ counters) {
    constexpr int NT = T * T < 256 ? T * T : 256;
    constexpr int PPT = T * T / NT;
    constexpr int ROWS = NT / T;
    __shared__ unsigned long long s_cnt[3];
    if (threadIdx.x < 3) s_cnt[threadIdx.x] = 0ull;
    __syncthreads();
    int v, ty, tx;
    ViewDesc vd;
    // the tiles and pixels the compositing kernels take (fovea-culled: the disk's)
    const bool valid = launch_tile(blockIdx.x, tm, views, nviews, T, v, vd, ty, tx) &&
                       (!tm.gaze || fovea_tile_live(tm.gaze, v, tm.radius, vd.width, vd.height, T, tx, ty));
    const float disk_r = cull_gaze ? cull_radius * (float)vd.width : 0.f;
    const uint2 rg = valid ? ranges[blockIdx.x] : make_uint2(0u, 0u);
    unsigned long long visit = 0, incl = 0, visit_bwd = 0;
#pragma unroll
    for (int k = 0; k < PPT; k++) {
        const int x = tx * T + threadIdx.x % T, y = ty * T + threadIdx.x / T + k * ROWS;
        if (!(x < vd.width && y < vd.height)) continue;
        if (!in_fovea(cull_gaze, v, x, y, disk_r)) continue;
        const float px = (float)x, py = (float)y;
        float Tr = 1.f;
        uint32_t last = 0;
        for (uint32_t e = rg.x; e < rg.y; e++) {
            const uint32_t r = vals[e];
            visit++;
            float alpha, ae, ex, dx, dy;
            const float4 *rr = sp.at(r, 0);
            const float4 ra = rr[kRecA], rb = rr[kRecB], c = rr[kRecC];
            if (!splat_alpha(ra, rb, c, px, py, alpha, ae, ex, dx, dy)) continue;
            const float Tn = Tr * (1.f - alpha);
            if (Tn < kTStop) break;
            Tr = Tn;
            incl++;
            last = e - rg.x + 1u;
        }
        visit_bwd += last;
    }
    atomicAdd(&s_cnt[0], visit);
    atomicAdd(&s_cnt[1], incl);
    atomicAdd(&s_cnt[2], visit_bwd);
    __syncthreads();
    if (threadIdx.x < 3) atomicAdd(&counters[threadIdx.x], s_cnt[threadIdx.x]);
}

__global__ void k_zero_u64(unsigned long long *p, int n) {
    if ((int)threadIdx.x < n) p[threadIdx.x] = 0ull;
}

// ---- loss -----------------------------------------------------------------------

constexpr int kLossBlock = 256;
constexpr int kLossPx = 4;                         // pixels per thread of a loss launch
constexpr int kLossSpan = kLossBlock * kLossPx;    // pixels per block

__device__ __forceinline__ int view_of_pixel(const ViewDesc *__restrict__ views, int nviews, uint32_t p) {
    int v = 0;
    while (v + 1 < nviews && p >= (uint32_t)views[v + 1].pix_off) v++;
    return v;
}


// Blocks per view of a fovea-window loss launch: each view's box x box window
// is covered by whole blocks, so a block's view is uniform.
__host__ __device__ __forceinline__ int loss_blocks_per_view(int box) {
    return (box * box + kLossSpan - 1) / kLossSpan;
}

// Pixel t (< kLossSpan) of block bi of a loss launch: every pixel of every view
// (box == 0: pixel bi kLossSpan + t), or in view bi / bpv the pixel
// (bi mod bpv) kLossSpan + t of its box x box window, which starts at its
// first fovea tile (fovea culling; false for window pixels outside the view or
// past its last fovea tile).  f: the view's fovea tiles (box mode, computed once
// per block by the caller).  Plans hold fewer than 2^31 pixels: 32-bit
// arithmetic.
__device__ __forceinline__ bool loss_pixel(uint32_t bi, uint32_t t, uint32_t total_pix, int box,
                                           int tile, const FoveaTiles &f,
                                           const ViewDesc *__restrict__ views, int nviews, int &v,
                                           int &x, int &y) {
    if (box == 0) {
        const uint32_t p = bi * kLossSpan + t;
        if (p >= total_pix) return false;
        v = view_of_pixel(views, nviews, p);
        const ViewDesc vd = views[v];
        const uint32_t q = p - (uint32_t)vd.pix_off;
        y = (int)(q / (uint32_t)vd.width);
        x = (int)(q - (uint32_t)y * (uint32_t)vd.width);
        return true;
    }
    const int bpv = loss_blocks_per_view(box);
    v = (int)(bi / (uint32_t)bpv);
    if (v >= nviews || f.tx0 > f.tx1) return false;
    const uint32_t l = (bi - (uint32_t)v * (uint32_t)bpv) * kLossSpan + t;
    if (l >= (uint32_t)(box * box)) return false;
    // l / box by a float reciprocal: exact, since l < 2^23 and box < 2^12 keep the
    // quotient's fraction at least 1 / (2 box) from an integer
    const uint32_t ly = (uint32_t)(((float)l + 0.5f) * __builtin_amdgcn_rcpf((float)box));
    x = f.tx0 * tile + (int)(l - ly * (uint32_t)box);
    y = f.ty0 * tile + (int)ly;
    const ViewDesc vd = views[v];
    return x < vd.width && y < vd.height && x < (f.tx1 + 1) * tile && y < (f.ty1 + 1) * tile;
}

// The fovea tiles of block bi's view (box mode), computed once per block.
__device__ __forceinline__ FoveaTiles block_fovea(uint32_t bi, int box, int tile,
                                                  const float *__restrict__ gaze, float radius_frac,
                                                  const ViewDesc *__restrict__ views, int nviews,
                                                  FoveaTiles *s_f) {
    __syncthreads();   // s_f of the previous block is no longer read
    if (threadIdx.x == 0) {
        FoveaTiles f{1, 0, 1, 0};
        const int v = box ? (int)(bi / (uint32_t)loss_blocks_per_view(box)) : 0;
        if (box && v < nviews) {
            const ViewDesc vd = views[v];
            f = fovea_tiles(gaze, v, radius_frac, vd.width, vd.height, tile);
        }
        *s_f = f;
    }
    __syncthreads();
    return *s_f;
}

// The masked entries, one thread per (view, row of the pixels the loss visits):
// every pixel of the view (box == 0) or of its box x box window from its first
// fovea tile, clipped to the view and to the fovea tiles (as loss_pixel).  On a
// row the mask is an interval: in_fovea compares fl(dx)^2 + dy^2 with r^2, where
// dx = fl(x + 0.5 - gaze_x), and rounding is monotone, so the test can only turn
// false as |x + 0.5 - gaze_x| grows.  The row's pixel nearest the gaze column
// decides whether it has any, and a binary search each way (on that same test)
// finds the ends: the count equals the pixel-by-pixel count exactly.
__global__ __launch_bounds__(kLossBlock) void k_loss_count(const float *__restrict__ gaze,
                                                           float radius_frac,
                                                           const ViewDesc *__restrict__ views,
                                                           int nviews, int rows, int box, int tile,
                                                           uint32_t channels,
                                                           uint32_t *__restrict__ mask_count) {
    __shared__ uint32_t s_red[kLossBlock / 64];
    const uint32_t i = blockIdx.x * kLossBlock + threadIdx.x;
    const int v = (int)(i / (uint32_t)rows);
    const int row = (int)(i - (uint32_t)v * (uint32_t)rows);
    uint32_t n = 0u;
    if (v < nviews) {
        const ViewDesc vd = views[v];
        int x0 = 0, x1 = vd.width - 1, y = row;
        bool ok = row < vd.height;
        if (box) {
            const FoveaTiles f = fovea_tiles(gaze, v, radius_frac, vd.width, vd.height, tile);
            x0 = f.tx0 * tile;
            x1 = min(min((f.tx1 + 1) * tile, vd.width), x0 + box) - 1;
            y = f.ty0 * tile + row;
            ok = f.tx0 <= f.tx1 && y < min((f.ty1 + 1) * tile, vd.height);
        }
        if (ok) {
            const float rad = radius_frac * (float)vd.width;
            // the row's pixel nearest the gaze column (fmaxf takes x0 for a NaN gaze)
            const int xm = (int)fminf(fmaxf(rintf(gaze[2 * v] - 0.5f), (float)x0), (float)x1);
            if (in_fovea(gaze, v, xm, y, rad)) {
                int lo = xm, hi = x1 + 1;   // in at lo, out at hi (or past the row)
                while (hi - lo > 1) {
                    const int mid = lo + (hi - lo) / 2;
                    if (in_fovea(gaze, v, mid, y, rad)) lo = mid;
                    else hi = mid;
                }
                const int xr = lo;
                lo = x0 - 1;   // out at lo (or before the row), in at hi
                hi = xm;
                while (hi - lo > 1) {
                    const int mid = lo + (hi - lo) / 2;
                    if (in_fovea(gaze, v, mid, y, rad)) hi = mid;
                    else lo = mid;
                }
                n = (uint32_t)(xr - hi + 1) * channels;
            }
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) n += (uint32_t)__shfl_xor((int)n, o, 64);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = n;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t tot = 0u;
#pragma unroll
        for (int w = 0; w < kLossBlock / 64; w++) tot += s_red[w];
        if (tot) atomicAdd(mask_count, tot);
    }
}

// Per-pixel L1 terms and sign gradient, and one partial sum per workgroup.
// The count of masked entries comes from mask_count (device) or count_host.
// (A last-workgroup-done reduction would need an agent-scope release fence per
// workgroup, which writes back the L2 just filled with dL/dRGBA; the sum is left
// to a workgroup of a later kernel.)
__global__ __launch_bounds__(kLossBlock) void k_loss_l1(
    const float *__restrict__ rgba, const float *__restrict__ target, const float *__restrict__ gaze,
    float radius_frac, const ViewDesc *__restrict__ views, int nviews, int64_t total_pix, int box,
    int tile, int tgt_planes, bool alpha_term, const float *__restrict__ bg,
    const uint32_t *__restrict__ mask_count, uint32_t count_host, float *__restrict__ dl,
    float *__restrict__ partial) {
    __shared__ float s_red[kLossBlock / 64];
    __shared__ FoveaTiles s_f;
    const uint32_t cnt = mask_count ? *mask_count : count_host;
    const FoveaTiles f = box ? block_fovea(blockIdx.x, box, tile, gaze, radius_frac, views, nviews, &s_f)
                             : FoveaTiles{1, 0, 1, 0};
    float s = 0.f;
    const float inv = 1.f / (float)max(cnt, 1u);
    // kLossPx pixels per thread, kLossBlock apart (each step coalesced); all
    // their loads are issued before any is used
    bool ok[kLossPx], in[kLossPx];
    int vk[kLossPx];
    uint32_t qk[kLossPx], plk[kLossPx], offk[kLossPx];
    if (box) {   // the block's view is uniform: its descriptor is read once
        const int vb = min((int)(blockIdx.x / (uint32_t)loss_blocks_per_view(box)), nviews - 1);
        const ViewDesc vd = views[vb];
        const float rad = radius_frac * (float)vd.width;
#pragma unroll
        for (int k = 0; k < kLossPx; k++) {
            int v = 0, x = 0, y = 0;
            ok[k] = loss_pixel(blockIdx.x, (uint32_t)(k * kLossBlock) + threadIdx.x, (uint32_t)total_pix,
                               box, tile, f, views, nviews, v, x, y);
            vk[k] = vb;
            qk[k] = (uint32_t)(y * vd.width + x);
            plk[k] = (uint32_t)vd.width * (uint32_t)vd.height;
            offk[k] = (uint32_t)vd.pix_off;
            in[k] = ok[k] && in_fovea(gaze, vb, x, y, rad);
        }
    } else {
#pragma unroll
        for (int k = 0; k < kLossPx; k++) {
            int v = 0, x = 0, y = 0;
            ok[k] = loss_pixel(blockIdx.x, (uint32_t)(k * kLossBlock) + threadIdx.x, (uint32_t)total_pix,
                               box, tile, f, views, nviews, v, x, y);
            const ViewDesc vd = views[ok[k] ? v : 0];
            vk[k] = v;
            qk[k] = (uint32_t)(y * vd.width + x);
            plk[k] = (uint32_t)vd.width * (uint32_t)vd.height;
            offk[k] = (uint32_t)vd.pix_off;
            in[k] = ok[k] && in_fovea(gaze, v, x, y, radius_frac * (float)vd.width);
        }
    }
    // RGBA targets: colour premultiplied, composited over the view background.
    // A pixel outside the mask reads nothing (a fovea-culled forward did not
    // composite it) and gets a zero gradient - written only on full frames:
    // after a fovea-culled forward (box > 0) the adjoint does not read it (no
    // splat reached the pixel).
    float im[kLossPx][4], tg[kLossPx][4], bk[kLossPx][3];
#pragma unroll
    for (int k = 0; k < kLossPx; k++) {
        const size_t plane = plk[k], q = qk[k];
        const float *img = rgba + 4 * (size_t)offk[k];
        const float *tgt = target + (size_t)tgt_planes * offk[k];
        if (in[k]) {
#pragma unroll
            for (int c = 0; c < 3; c++) {
                im[k][c] = img[c * plane + q];
                tg[k][c] = tgt[c * plane + q];
            }
            im[k][3] = alpha_term ? img[3 * plane + q] : 0.f;
            tg[k][3] = tgt_planes == 4 || alpha_term ? tgt[3 * plane + q] : 1.f;
            if (bg) {
#pragma unroll
                for (int c = 0; c < 3; c++) bk[k][c] = bg[3 * vk[k] + c];
            }
        }
    }
#pragma unroll
    for (int k = 0; k < kLossPx; k++) {
        if (!(ok[k] && (in[k] || !box))) continue;
        const size_t plane = plk[k], q = qk[k];
        float *g = dl + 4 * (size_t)offk[k];
        const float ta = in[k] && tgt_planes == 4 ? tg[k][3] : 1.f;
#pragma unroll
        for (int c = 0; c < 4; c++) {
            float gv = 0.f;
            if (in[k] && (c < 3 || alpha_term)) {
                float t = tg[k][c];
                if (c < 3 && bg) t = fmaf(1.f - ta, bk[k][c], t);
                const float d = im[k][c] - t;
                s += fabsf(d);
                gv = d > 0.f ? inv : (d < 0.f ? -inv : 0.f);
            }
            g[c * plane + q] = gv;
        }
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) s += __shfl_xor(s, o, 64);   // fixed tree: deterministic
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        float tot = 0.f;
#pragma unroll
        for (int w = 0; w < kLossBlock / 64; w++) tot += s_red[w];
        partial[blockIdx.x] = tot;
    }
}

// One workgroup for the loss's final reduction (loss_tail).
__global__ __launch_bounds__(1024) void k_loss_final(LossTail lt) {
    __shared__ float s_part[kTailWaves];
    loss_tail<kTailWaves>(lt, s_part);
}

// Per-view random background: SplitMix64 (Steele, Lea and Flood, OOPSLA 2014)
// output k = 1 + (step * kMaxViews + v) * 4 + c from state seed, i.e. the
// state seed + k * golden-ratio increment passed through the published
// finaliser; the top 24 bits scaled to [0, 1) (exact in float).
__global__ void k_draw_bg(uint64_t seed, const int32_t *__restrict__ step, int nviews,
                          float *__restrict__ bg) {
    const int e = threadIdx.x;
    if (e >= 3 * nviews) return;
    const int v = e / 3, c = e - 3 * v;
    const uint64_t k = 1ull + ((uint64_t)step[0] * kMaxViews + (uint64_t)v) * 4ull + (uint64_t)c;
    uint64_t z = seed + k * 0x9E3779B97F4A7C15ull;
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    z ^= z >> 31;
    bg[e] = (float)(uint32_t)(z >> 40) * (1.f / 16777216.f);
}

__global__ void k_fill_u32(uint32_t *p, int64_t n, uint32_t value) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        p[e] = value;
}

__global__ void k_fill_f32(float *p, int64_t n, float value) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n;
         e += (int64_t)gridDim.x * blockDim.x)
        p[e] = value;
}

template <int T, int B, bool SPLIT>
void render_fwd_tbs(hipStream_t s, const RenderArgs &a, float *out) {
    constexpr int NT = fwd_threads<T, SPLIT>();
    const int g = SPLIT ? 4 * ((a.total_tiles + 7) / 8 * 8) : a.total_tiles;
    if (a.t_mode == 1)
        k_render_fwd<T, B, 1, SPLIT><<<g, NT, 0, s>>>(a.order, a.ranges, a.vals, a.sp, a.views,
                                                     a.nviews, a.cams, out, a.tfinal, a.ncontrib, a.ckpt,
                                                     a.fstate, nullptr, a.bg, a.cull_gaze, a.cull_radius,
                                                     a.total_tiles, a.tm);
    else if (a.t_mode == 2)
        k_render_fwd<T, B, 2, SPLIT><<<g, NT, 0, s>>>(a.order, a.ranges, a.vals, a.sp, a.views,
                                                     a.nviews, a.cams, out, a.tfinal, a.ncontrib, nullptr,
                                                     nullptr, a.tstore, a.bg, a.cull_gaze, a.cull_radius,
                                                     a.total_tiles, a.tm);
    else
        k_render_fwd<T, B, 0, SPLIT><<<g, NT, 0, s>>>(a.order, a.ranges, a.vals, a.sp, a.views,
                                                     a.nviews, a.cams, out, a.tfinal, a.ncontrib, nullptr,
                                                     nullptr, nullptr, a.bg, a.cull_gaze, a.cull_radius,
                                                     a.total_tiles, a.tm);
}

// Split 16-pixel tiles into one workgroup per quadrant when the plan has at
// most kSplitTilesPerCu tiles per compute unit: measured on one 1024^2 view
// (4096 tiles) it shortens the forward by 5%, on 16 views of 1920^2 (230k
// tiles) it lengthens it by 2.5% and on 8 views of 0.25-4 Mpix (63k tiles)
// by 6-18%.
constexpr int kSplitTilesPerCu = 16;

template <int T, int B>
void render_fwd_tb(hipStream_t s, const RenderArgs &a, float *out) {
    if (T == 16 && (int64_t)a.total_tiles <= (int64_t)kSplitTilesPerCu * a.cus)
        render_fwd_tbs<T, B, T == 16>(s, a, out);
    else
        render_fwd_tbs<T, B, false>(s, a, out);
}

template <int T, bool WIDE>
void render_bwd_tw(hipStream_t s, const RenderArgs &a, const float *dl) {
    constexpr int NT = adj_threads<T, WIDE>();
    const int tail = a.tail.partial ? 1 : 0;
    if (a.t_mode == 1)
        k_render_bwd_ckpt<T, WIDE><<<a.bwd_grid + tail, NT, 0, s>>>(
            a.ranges, a.total_tiles, (uint32_t)a.batch, a.m_dev, a.m_host, a.vals, a.sp, a.views, a.nviews,
            a.cams, a.tfinal, a.ncontrib, a.fstate, a.ckpt, a.bg, dl, a.kp, a.tm, a.tail);
    else if (a.t_mode == 2)
        k_render_bwd<T, 2, WIDE><<<a.total_tiles + tail, NT, 0, s>>>(a.order, a.ranges, a.vals, a.sp, a.views,
                                                             a.nviews, a.cams, a.tfinal, a.ncontrib,
                                                             a.tstore, a.bg, dl, a.kp, a.tm, a.tail);
    else
        k_render_bwd<T, 0, WIDE><<<a.total_tiles + tail, NT, 0, s>>>(a.order, a.ranges, a.vals, a.sp, a.views,
                                                             a.nviews, a.cams, a.tfinal, a.ncontrib,
                                                             nullptr, a.bg, dl, a.kp, a.tm, a.tail);
}

template <int T>
void render_fwd_t(hipStream_t s, const RenderArgs &a, float *out) {
    if (a.batch == 64) render_fwd_tb<T, 64>(s, a, out);
    else if (a.batch == 128) render_fwd_tb<T, 128>(s, a, out);
    else render_fwd_tb<T, 256>(s, a, out);
}

// The adjoint takes one wave per 8 x 8 block while the plan has at most
// kWideTilesPerCu (checkpointed mode, whose units cut the lists short:
// kWideCkptTilesPerCu) 16-pixel tiles' worth of tiles per compute unit, one wave per
// tile above.  Fit steps with blocks against tiles, 20,000 phantom and 30,000 random
// Gaussians: recomputed on 512^2 276 : 471 and 199 : 283 us, on 800^2 222 : 346 and
// 230 : 258, on 1024^2 218 : 312 and 285 : 270; checkpointed on 256^2 224 : 237 and 181 :
// 180, on 384^2 170 : 185 and 176 : 171, on 512^2 171 : 170 and 203 : 176.  An 8-pixel
// tile is one block and has one wave in both forms: there the products only cost.
constexpr int kWideTilesPerCu = 16, kWideCkptTilesPerCu = 3;

template <int T>
void render_bwd_t(hipStream_t s, const RenderArgs &a, const float *dl) {
    const int per_cu = a.t_mode == 1 ? kWideCkptTilesPerCu : kWideTilesPerCu;
    if constexpr (T > 8) {
        if ((int64_t)a.total_tiles * (T * T) <= (int64_t)per_cu * 256 * a.cus) {
            render_bwd_tw<T, true>(s, a, dl);
            return;
        }
    }
    render_bwd_tw<T, false>(s, a, dl);
}

}  // namespace

void launch_render_fwd(hipStream_t s, const RenderArgs &a, float *out_rgba) {
    if (a.tile == 8) render_fwd_t<8>(s, a, out_rgba);
    else if (a.tile == 16) render_fwd_t<16>(s, a, out_rgba);
    else render_fwd_t<32>(s, a, out_rgba);
}

void launch_render_bwd(hipStream_t s, const RenderArgs &a, const float *dl_drgba) {
    if (a.tile == 8) render_bwd_t<8>(s, a, dl_drgba);
    else if (a.tile == 16) render_bwd_t<16>(s, a, dl_drgba);
    else render_bwd_t<32>(s, a, dl_drgba);
}

void launch_grad_sum(hipStream_t s, const KeyPlace &kp, int nrec, float *g2d) {
    if (nrec <= 0) return;
    k_grad_sum<<<(nrec + 63) / 64, 64, 0, s>>>(kp, nrec, g2d);
}

void launch_count_pairs(hipStream_t s, int tile, int total_tiles, const uint2 *ranges,
                        const uint32_t *vals, SplatPtrs sp, const ViewDesc *views, int nviews,
                        const TileMap &tm, const float *cull_gaze, float cull_radius,
                        unsigned long long *counters) {
    k_zero_u64<<<1, 64, 0, s>>>(counters, 3);
    if (tile == 8)
        k_count_pairs<8><<<total_tiles, 64, 0, s>>>(ranges, vals, sp, views, nviews, tm, cull_gaze, cull_radius, counters);
    else if (tile == 16)
        k_count_pairs<16><<<total_tiles, 256, 0, s>>>(ranges, vals, sp, views, nviews, tm, cull_gaze, cull_radius, counters);
    else
        k_count_pairs<32><<<total_tiles, 256, 0, s>>>(ranges, vals, sp, views, nviews, tm, cull_gaze, cull_radius, counters);
}

// Partial sums of a loss launch: one per block (a fovea-window launch's views
// are padded to whole blocks, at most one more block per view).
int loss_partials(int64_t total_pix) {
    return (int)((total_pix + kLossBlock - 1) / kLossBlock) + kMaxViews;
}

int loss_launch_blocks(int64_t total_pix, int nviews, int box) {
    return box ? nviews * loss_blocks_per_view(box) : (int)((total_pix + kLossSpan - 1) / kLossSpan);
}

LossTail launch_loss_l1(hipStream_t s, const float *rgba, const float *target, const float *gaze,
                    float radius_frac, const ViewDesc *views, int nviews, int64_t total_pix,
                    float *dl, float *partial, uint32_t *mask_count, float *loss, uint32_t *flags,
                    int32_t *step_inc, int box, int tile, int tgt_planes, bool alpha_term,
                    const float *bg, uint32_t norm_count, bool accumulate, int max_height, bool defer) {
    if (!gaze) box = 0;
    const uint32_t channels = alpha_term ? 4u : 3u;
    const int nb = loss_launch_blocks(total_pix, nviews, box);
    if (gaze && norm_count == 0u)
        launch_loss_count(s, gaze, radius_frac, views, nviews, max_height, box, tile, channels,
                          mask_count);
    const uint32_t *mc = gaze && norm_count == 0u ? mask_count : nullptr;
    const uint32_t cnt = norm_count ? norm_count : (uint32_t)(channels * total_pix);
    k_loss_l1<<<nb, kLossBlock, 0, s>>>(rgba, target, gaze, radius_frac, views, nviews, total_pix, box,
                                        tile, tgt_planes, alpha_term, bg, mc, cnt, dl, partial);
    const LossTail lt{partial, nb, mc, cnt, loss, flags, step_inc, accumulate};
    if (!defer) k_loss_final<<<1, 64 * kTailWaves, 0, s>>>(lt);
    return lt;
}

void launch_loss_count(hipStream_t s, const float *gaze, float radius_frac, const ViewDesc *views,
                       int nviews, int max_height, int box, int tile, uint32_t channels,
                       uint32_t *mask_count) {
    const int rows = box ? box : max_height;
    const int64_t threads = (int64_t)nviews * rows;
    k_fill_u32<<<1, 64, 0, s>>>(mask_count, 1, 0u);
    if (threads > 0)
        k_loss_count<<<(int)((threads + kLossBlock - 1) / kLossBlock), kLossBlock, 0, s>>>(
            gaze, radius_frac, views, nviews, rows, box, tile, channels, mask_count);
}

void launch_draw_bg(hipStream_t s, uint64_t seed, const int32_t *step, int nviews, float *bg) {
    k_draw_bg<<<1, 3 * kMaxViews, 0, s>>>(seed, step, nviews, bg);
}

void launch_fill_u32(hipStream_t s, uint32_t *p, int64_t n, uint32_t value) {
    if (n <= 0) return;
    int64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    k_fill_u32<<<(int)g, 256, 0, s>>>(p, n, value);
}

void launch_fill_f32(hipStream_t s, float *p, int64_t n, float value) {
    if (n <= 0) return;
    int64_t g = (n + 255) / 256;
    if (g > 4096) g = 4096;
    k_fill_f32<<<(int)g, 256, 0, s>>>(p, n, value);
}

}  // namespace gsf
