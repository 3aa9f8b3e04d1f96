// gsr_composite.hip -- per-tile compositing on gfx950 (A6 forward, A7 backward).
//
// Mapping.  A tile is 16 pixels wide and a multiple of 4 high; a "slab" is 16
// x 4 of its pixels, one per lane of a wave64 (lane l: column l % 16, row
// l / 16).  W waves share a tile, each owning RPL consecutive slabs (pixel
// state in registers, RPL pixels per lane).  A tile's sorted list is consumed
// in batches of 64 W records: each thread stages one record in LDS (pre-scaled
// conic, tile-relative centre, and the mask of the slabs its alpha >= 1/255
// ellipse reaches), then every wave lists the records that meet its slabs by
// a ballot over the masks and walks that list four records at a time in
// straight-line code, reading them back as LDS broadcasts.  So a record costs
// a wave nothing where it misses its slabs, four exponentials are in flight
// before the transmittance chain needs the first, and no row tests whether it
// is worth evaluating (all but about 5 % of the listed ones are).  The pixel
// updates are branch-free (selects and the execution mask).  Against one record at
// a time with a skip test per row, one wave per tile, this took the fused step of
// a 1080p view of 1M Gaussians from 332 to 303 us and of 200k from 265 to 224 us.
//
// Waves per tile.  One wave per tile leaves the chip idle when a call has few
// tiles, each a serial chain over its list: 640 x 480 has 1,200 tiles of 16 x
// 16 for 1,024 SIMDs.  W > 1 splits the chain (forward 77 -> 26 us, backward
// 123 -> 48 us there, W = 4), but repeats the records' part of the work in
// every wave and, in the backward, the reduction; tile_waves() has the rule.
// The image does not depend on W (each pixel's arithmetic and order are the
// same); the moments are summed in another order.
//
// Early stop.  Dense scenes saturate long before the end of a tile's list: a
// wave drops a slab once all its pixels have stopped, and the forward records
// per tile the number of list positions any of its pixels used (nmax).  The
// backward replays only [start, start + nmax) and flags the pair slots whose
// moments it writes; the per-Gaussian reduction reads those only.
//
// Backward.  Front to back again (nothing per (pixel, Gaussian) is stored):
// from the forward's output C_out and the running accumulation, the colour
// behind contributor k is B_k = C_out - sum_{j<=k} c_j a_j T_j; only its
// projection on the upstream gradient g is needed, kept as one running value
// g.B = g.C_out - sum, from which alpha dL/dalpha = w g.c - g.B alpha / (1 - alpha)
// (w = alpha T); with g.B taken after the Gaussian's own term and
// T' = T (1 - alpha) that is w (g.c - g.B / T'), one reciprocal per row and
// one fused multiply-add for the update of g.B.
// Per pair the kernel produces nine moments over the tile's pixels: with
// w = dL/dsigma, the sums of w dx, w dy, w dx^2, w dx dy, w dy^2, of
// alpha dL/dalpha and of the colour gradient; they are linear in the per-pixel
// terms, so the conversion to (u, v, conic, opacity) gradients happens once
// per Gaussian after the reduction over its tiles.
//
// Reduction.  A lane's column fixes dx, so the lanes of one column (the four
// rows of 16 lanes) only need the sums of six values: sa = alpha dL/dalpha,
// sa dy, sa dy^2 and the colour gradient.  For four Gaussians together two
// lane-swap levels (v_permlane32_swap, v_permlane16_swap: two instructions
// turn two values into one register of half sums) leave six registers whose
// row q holds Gaussian q's 16 column sums; the products with dx follow, once
// for all four, and 36 lanes add the 16 columns of one (Gaussian, moment)
// each from LDS, in a fixed order (no atomics, deterministic).  About 16
// instructions per Gaussian, against 30 for nine values summed over lane
// quads and transposed through LDS.  With W > 1 the waves' moments of 64
// records are added in wave order before they are written.
//
// Values that are not finite.  A listed record need not reach every pixel of a
// slab, or any, so what the backward adds for it is kept from the other pixels by
// their mask, not by a factor of 0: an upstream gradient that is not finite
// spoils the gradients of the Gaussians that composite on its pixel, and of no
// others.  (The steps of one view cost up
// to 0.5 % for it: 70.5 against 70.2 us at 128 x 128, 428 against 426 us at
// 720p, 520 against 521 us at 1080p with 1M Gaussians.)  An exponent
// that is not a number reaches no pixel, and an infinite colour the pixels that
// its Gaussian composites on (the records hold it as a large one).
//
// Schedule.  The forward files every tile in a bucket of its replay count
// (nmax), and the backward's workgroups take the tiles heaviest first: in
// tile order the dense centre tiles, dispatched late, left a tail.  Which
// workgroup takes which tile changes no result.
//
// Fused step.  For the mean absolute error the upstream gradient of a pixel
// is a function of that pixel's colour alone, so the fused pass runs a tile's
// forward and, in the same workgroup, its backward: the same device
// functions, so the results are theirs bit for bit, but a SIMD then holds
// waves in both phases (the backward's arithmetic fills the forward's
// latency), the forward's per-pixel state never leaves registers, and a list
// that fits one batch is staged once.  Its schedule cannot use this step's
// replay counts, which exist only after the forward; it takes the tile's list
// length, capped by the replay count the workspace holds from the previous
// step (exact for a repeated step, the list length on a fresh workspace).
#include "gsr_internal.h"

namespace gsr {

struct TileCtx {
    int v;
    uint32_t ox, oy;          // tile origin in pixels
    uint32_t width, height;   // view size
    uint32_t pix_off;         // first pixel of the view
    uint32_t tx, ty;          // tile coordinates
};

__device__ __forceinline__ TileCtx tile_ctx(const ViewTable &vt, uint32_t t) {
    int v = 0;
    while (v + 1 < vt.n_views && t >= vt.v[v + 1].tile_off) ++v;
    TileCtx c;
    c.v = v;
    const uint32_t lt = t - vt.v[v].tile_off;
    const uint32_t tx_n = (uint32_t)vt.v[v].tiles_x;
    c.tx = lt % tx_n;
    c.ty = lt / tx_n;
    c.ox = c.tx * kTileW;
    c.oy = c.ty * (uint32_t)vt.tile_h;
    c.width = (uint32_t)vt.v[v].width;
    c.height = (uint32_t)vt.v[v].height;
    c.pix_off = vt.v[v].pix_off;
    return c;
}

// Rows [y0, y1] of the tile (tile-relative pixel rows) narrowed to those that
// the Gaussian's alpha >= 1/255 ellipse reaches within the tile's columns.
// With (dx, dy) = pixel - centre and sigma = A dx^2 / 2 + B dx dy + C dy^2 / 2,
// the ellipse sigma <= s over the column band dx in [lo, hi] spans
// dy in [min h, max g] with g, h = (-B dx +- sqrt(2 C s - det dx^2)) / C,
// det = A C - B^2: g is concave with its peak at dx = -B sqrt(2 s / (A det)),
// h convex with its trough at the opposite dx, so each extreme is at that
// point clamped to the band.  FP32 with slack: s = 1.001 (ln(255 o) + 0.01)
// + 0.01 (the 1.001 grows the extents by far more than the evaluation's
// rounding, about 1e-6 relative, at any scale) and 0.01 px more on each
// side; a row left out then has alpha below 0.99 / 255 at every pixel, which
// the compositing's own FP32 evaluation cannot round up to 1/255, so leaving
// it out changes nothing but the work.  Degenerate conics keep the box's rows.
__device__ __forceinline__ void ellipse_rows_in_band(float A, float B, float C, float opacity, float ut, float vt,
                                                     int &y0, int &y1) {
    if (y0 > y1) return;
    const float det = A * C - B * B;
    const float s = 1.001f * (__logf(255.f * opacity) + 0.01f) + 0.01f;
    if (!(det > 0.f) || !(A > 0.f) || !(C > 0.f) || !(s > 0.f)) return;
    const float idet = __builtin_amdgcn_rcpf(det), iC = __builtin_amdgcn_rcpf(C);
    const float X = __builtin_sqrtf(2.f * C * s * idet);  // half-width of the ellipse
    const float lo = fmaxf(0.5f - ut - 0.01f, -X), hi = fminf((float)kTileW - 0.5f - ut + 0.01f, X);
    if (lo > hi) {  // the ellipse misses the tile's columns
        y1 = y0 - 1;
        return;
    }
    const float xs = -B * __builtin_sqrtf(2.f * s * idet * __builtin_amdgcn_rcpf(A));
    const float xt = fminf(fmaxf(xs, lo), hi), xb = fminf(fmaxf(-xs, lo), hi);
    const float top = (-B * xt + __builtin_sqrtf(fmaxf(0.f, 2.f * C * s - det * xt * xt))) * iC;
    const float bot = (-B * xb - __builtin_sqrtf(fmaxf(0.f, 2.f * C * s - det * xb * xb))) * iC;
    // pixel row r (centre r + 0.5) lies in [vt + bot, vt + top]
    const float r0 = ceilf(vt + bot - 0.51f), r1 = floorf(vt + top - 0.49f);
    y0 = max(y0, (int)fmaxf(r0, -1.f));
    y1 = min(y1, (int)fminf(r1, 65536.f));
}

// Staged record (LDS): three float4 per Gaussian.
//   a = (u - ox, v - oy, -A log2e / 2, -B log2e)
//   b = (-C log2e / 2, log2(opacity), red, green)
//   d = (blue, bits(slab mask), bits(pair index), opacity)
// so that sigma * log2e = -(a.z dx^2 + a.w dx dy + b.x dy^2) and
// alpha = min(0.99, exp2(-sigma log2e + b.y)).  Bit k of the slab mask is set
// when the Gaussian's alpha >= 1/255 ellipse (with slack) reaches rows
// [4k, 4k + 3] of the tile within its columns.
__device__ __forceinline__ void stage_record(const Rec &r, uint32_t first_pair, const TileCtx &c, uint32_t tile_h,
                                             float4 &a, float4 &b, float4 &d) {
    const float ut = (r.r0.x - (float)c.ox) + r.r3.x;
    const float vt = (r.r0.y - (float)c.oy) + r.r3.y;
    a = make_float4(ut, vt, -0.5f * kLog2e * r.r0.z, -kLog2e * r.r0.w);
    b = make_float4(-0.5f * kLog2e * r.r1.x, __log2f(r.r1.y), r.r1.z, r.r1.w);
    const uint32_t by = __float_as_uint(r.r2.z);
    int y0 = max((int)(by & 0xffffu) - (int)c.oy, 0), y1 = min((int)(by >> 16) - (int)c.oy, (int)tile_h - 1);
    ellipse_rows_in_band(r.r0.z, r.r0.w, r.r1.x, r.r1.y, ut, vt, y0, y1);
    const uint32_t smask = y0 <= y1 ? ((2u << (y1 >> 2)) - 1u) & ~((1u << (y0 >> 2)) - 1u) : 0u;
    // pair index in emission order: offset + row-major position in the tile box
    const uint32_t bx = __float_as_uint(r.r2.y);
    const uint32_t tx0 = (bx & 0xffffu) / kTileW, tx1 = (bx >> 16) / kTileW;
    const uint32_t ty0 = (by & 0xffffu) / tile_h;
    const uint32_t p = first_pair + (c.ty - ty0) * (tx1 - tx0 + 1) + (c.tx - tx0);
    d = make_float4(r.r2.x, __uint_as_float(smask), __uint_as_float(p), r.r1.y);
}

// The slab mask of a staged record, as a scalar (the record is an LDS broadcast).
__device__ __forceinline__ uint32_t slab_mask(float packed) {
    return __builtin_amdgcn_readfirstlane(__float_as_uint(packed));
}

// The r-th tile of the backward's schedule: tiles in descending cost buckets
// (any order within a bucket: tiles are independent, so results do not
// depend on it), or tile r when the buckets do not hold every tile (a forward
// that skipped compositing).  One whole wave calls it.  Not inlined: its
// loop-invariant loads would otherwise be hoisted and held in registers
// through the tile's loops (13 more VGPRs, one wave fewer per SIMD).
__device__ __noinline__ uint32_t tile_by_cost(const uint32_t *__restrict__ order, uint32_t total_tiles,
                                                 uint32_t r) {
    const int lane = threadIdx.x & 63;
    static_assert(kCostBuckets == 2 * kWave, "two buckets per lane");
    // lane l: buckets 127 - 2l and 126 - 2l (descending cost)
    const uint32_t b0 = kCostBuckets - 1 - 2 * lane, c0 = order[b0], c1 = order[b0 - 1];
    const uint32_t incl = wave_inclusive_scan(c0 + c1, [](uint32_t a, uint32_t b) { return a + b; });
    if ((uint32_t)__shfl((int)incl, 63, 64) != total_tiles) return r;
    const unsigned long long past = __ballot(r < incl);  // lanes whose buckets end beyond r
    const int L = __ffsll((long long)past) - 1;
    const uint32_t before = (uint32_t)__shfl((int)(incl - c0 - c1), L, 64);
    const uint32_t cL0 = (uint32_t)__shfl((int)c0, L, 64);
    const uint32_t k = r - before;
    const uint32_t b = k < cL0 ? kCostBuckets - 1 - 2 * (uint32_t)L : kCostBuckets - 2 - 2 * (uint32_t)L;
    return order[kCostBuckets + (size_t)b * total_tiles + (k < cL0 ? k : k - cL0)];
}

// Exponent of alpha before the clamp, ex = log2(opacity) - sigma log2e
// = b.y + a.z dx^2 + a.w dx dy + b.x dy^2, for the pixel at (dx, dy) from the
// centre.  A lane's pixels share dx, so the dx terms and b.y are formed once
// per Gaussian (RowQuad) and each row evaluates (b.x dy + a.w dx) dy +
// (a.z dx^2 + b.y) by two fused multiply-adds.  sigma is a positive definite
// quadratic form (the conic inverts a covariance with the 0.3 I low-pass
// added), so there is no sign test: an FP32 exponent above b.y is rounding
// near the centre, where the exact sigma is >= 0 and the Gaussian counts.
struct RowQuad {
    float p, q;  // a.z dx^2 + b.y, a.w dx
};
__device__ __forceinline__ RowQuad row_quad(const float4 &a, const float4 &b, float dx) {
    return RowQuad{fmaf(a.z * dx, dx, b.y), a.w * dx};
}
__device__ __forceinline__ float alpha_exponent(const RowQuad &rq, const float4 &b, float dy) {
    return fmaf(fmaf(b.x, dy, rq.q), dy, rq.p);
}

// Alpha before the clamp to 0.99: exp2(ex), and 0 where that is not a number (of
// which the clamp would make 0.99).  The median with 0 and 1 is a modifier of the
// instruction, and what it cuts off the clamp would too.
__device__ __forceinline__ float raw_alpha(float ex) {
    return __builtin_amdgcn_fmed3f(__builtin_amdgcn_exp2f(ex), 0.f, 1.f);
}

// Zero gradient rows of the Gaussians of tile t's slice that no view saw, one
// row per lane (fire-and-forget stores that overlap the tile's ALU work).
__device__ __forceinline__ void zero_unseen_rows(const ZeroRows &z, uint32_t t, bool overflow, int lane,
                                                 int threads = kWave) {
    const uint64_t g0 = (uint64_t)t * z.per_tile, g1 = min(z.n, g0 + z.per_tile);
    const int K3 = 3 * z.sh_k;
    for (uint64_t i = g0 + (uint64_t)lane; i < g1; i += (uint64_t)threads) {
        bool seen = false;
        if (!overflow)
            for (int v = 0; v < z.n_views; ++v) seen |= z.count[(uint64_t)v * z.n + i] > 0u;
        if (seen) continue;
        for (int a = 0; a < 3; ++a) z.g.means[3 * i + a] = 0.f, z.g.log_scales[3 * i + a] = 0.f;
        reinterpret_cast<float4 *>(z.g.quats)[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        z.g.opacities[i] = 0.f;
        if ((K3 & 3) == 0) {
            float4 *row = reinterpret_cast<float4 *>(z.g.sh + (uint64_t)K3 * i);
            for (int k = 0; k < K3 / 4; ++k) row[k] = make_float4(0.f, 0.f, 0.f, 0.f);
        } else {
            float *row = z.g.sh + (uint64_t)K3 * i;
            for (int k = 0; k < K3; ++k) row[k] = 0.f;
        }
    }
}

__device__ __forceinline__ float l1_grad(float c, float target, float scale) {
    return c > target ? scale : (c < target ? -scale : 0.f);
}

// Slabs the forward walks together.  Two share a record's LDS reads and its
// dx terms but evaluate both where only one is met: faster for the four of a
// 16 x 16 tile's single wave (fused step of a 1080p view: 303 against 317 us),
// slower for two or eight (412 against 421 us, 1178 against 1243 us).
__host__ __device__ constexpr int forward_slabs(int rpl) { return rpl == 4 ? 2 : 1; }

constexpr int kGroup = 4;              // records per straight-line group
constexpr int kRedStride = kWave + 4;   // floats between two moments' rows (spreads the 16-byte reads over banks)

template <int W>
struct Staged {
    float4 a[W * kWave + 1], b[W * kWave + 1], d[W * kWave + 1];  // the last record never contributes
    uint32_t any[W];
};
template <int W>
struct Reduce {
    alignas(16) float red[W][kPartialStride * kRedStride];
    float mom[W > 1 ? W : 1][W > 1 ? kWave * kPartialStride : 1];
    unsigned long long live[W];
};

// Stages the list positions [b0, b0 + 64 W) below `end` (slab mask 0 beyond it).
template <int W>
__device__ __forceinline__ void stage_batch(Staged<W> &sh, const ViewTable &vt, const TileCtx &c, uint32_t b0,
                                            uint32_t end, const uint32_t *__restrict__ pval,
                                            const Rec *__restrict__ rec, const uint32_t *__restrict__ ioff) {
    const uint32_t tid = threadIdx.x, idx = b0 + tid;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f), b = a, d = a;
    if (idx < end) {
        const uint32_t item = pval[idx];
        stage_record(rec[item], ioff ? ioff[item] : 0u, c, (uint32_t)vt.tile_h, a, b, d);
    }
    sh.a[tid] = a;
    sh.b[tid] = b;
    sh.d[tid] = d;
}

// The record that never contributes (exponent -1000 everywhere).
template <int W>
__device__ __forceinline__ void stage_sentinel(Staged<W> &sh) {
    if (threadIdx.x == 0) {
        sh.a[W * kWave] = sh.d[W * kWave] = make_float4(0.f, 0.f, 0.f, 0.f);
        sh.b[W * kWave] = make_float4(0.f, -1000.f, 0.f, 0.f);
    }
}

// Takes the next kGroup records off the list m (a bit per record of the
// staged sub-batch s): their staged indices, the sentinel's once the list is
// empty; `packed` holds their positions in the sub-batch, a byte each.
// Returns how many are real.
template <int W>
__device__ __forceinline__ int take_group(unsigned long long &m, int s, int (&j)[kGroup], uint32_t &packed) {
    int n = 0;
    packed = 0u;
#pragma unroll
    for (int q = 0; q < kGroup; ++q) {
        const bool on = m != 0ull;
        const int l = on ? (int)__builtin_ctzll(m) : 0;
        j[q] = on ? s * kWave + l : W * kWave;
        packed |= (uint32_t)l << (8 * q);
        m &= m - 1ull;  // (stays 0)
        n += on ? 1 : 0;
    }
    return n;
}

// Forward over the records listed in m for KP slabs of the wave.  Returns
// whether some pixel of them still composites.
template <int KP, int W, bool STATS>
__device__ __forceinline__ bool forward_list(const Staged<W> &sh, unsigned long long m, int s, uint32_t pos0, float pxl,
                                             float pyl, float *T, float *C0, float *C1, float *C2, uint32_t *last,
                                             uint32_t *ncontrib, uint32_t *stop_at) {
    bool go = true;
    while (m) {
        int j[kGroup];
        uint32_t packed;
        take_group<W>(m, s, j, packed);
        float4 b[kGroup];
        float blue[kGroup], al[kGroup][KP];
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            const float4 a = sh.a[j[q]];
            b[q] = sh.b[j[q]];
            blue[q] = sh.d[j[q]].x;
            const RowQuad rq = row_quad(a, b[q], a.x - pxl);
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const float dy = a.y - (pyl + (float)(4 * k));
                al[q][k] = fminf(kAlphaMax, raw_alpha(alpha_exponent(rq, b[q], dy)));
            }
        }
#pragma unroll
        for (int q = 0; q < kGroup; ++q) {
            const uint32_t pos = pos0 + (uint32_t)j[q];
#pragma unroll
            for (int k = 0; k < KP; ++k) {
                const bool ok = al[q][k] >= kAlphaMin;
                const float wa = al[q][k] * T[k];
                const float Tn = T[k] - wa;  // T (1 - alpha)
                // a stopped pixel has Tn <= 0 < kTMin, so it never adds again; the
                // pixel stops where ok holds and add does not
                const bool add = ok & (Tn >= kTMin);
                const float w = add ? wa : 0.f;
                C0[k] = fmaf(b[q].z, w, C0[k]);
                C1[k] = fmaf(b[q].w, w, C1[k]);
                C2[k] = fmaf(blue[q], w, C2[k]);
                last[k] = add ? pos + 1 : last[k];
                if constexpr (STATS) {
                    ncontrib[k] += add ? 1u : 0u;
                    stop_at[k] = (ok && !add && T[k] > 0.f) ? pos : stop_at[k];
                }
                const float Ts = ok ? -fabsf(T[k]) : T[k];
                T[k] = add ? Tn : Ts;
            }
        }
        bool any = false;
#pragma unroll
        for (int k = 0; k < KP; ++k) any |= T[k] > 0.f;
        go = __ballot(any) != 0ull;
        if (!go) break;
    }
    return go;
}

// A6 for one tile: the wave's RPL slabs over the tile's sorted list, from the
// per-pixel state (T > 0: still compositing; T < 0: stopped, or outside the
// image, and -T is the final transmittance) to the colours and, per pixel, the
// list position after its last contributor.  `staged`: the first position of
// the batch left in LDS.
template <int RPL, int W, int KP, bool STATS>
__device__ __forceinline__ void tile_forward(Staged<W> &sh, const ViewTable &vt, const TileCtx &c, uint2 rg,
                                             const uint32_t *__restrict__ pval, const Rec *__restrict__ rec,
                                             const uint32_t *__restrict__ ioff, int wave, int lane, float pxl, float pyl,
                                             float (&T)[RPL], float (&C0)[RPL], float (&C1)[RPL], float (&C2)[RPL],
                                             uint32_t (&last)[RPL], uint32_t (&ncontrib)[RPL],
                                             uint32_t (&stop_at)[RPL], uint32_t &staged) {
    static_assert(RPL % KP == 0, "whole passes");
    stage_sentinel(sh);
    uint32_t alive = 0;  // passes with a pixel still compositing (wave-uniform)
#pragma unroll
    for (int k = 0; k < RPL; ++k) alive |= __ballot(T[k] > 0.f) != 0ull ? 1u << (k / KP) : 0u;
    for (uint32_t b0 = rg.x; b0 < rg.y; b0 += W * kWave) {
        if (b0 != rg.x) {  // leave once every wave's pixels have stopped
            if constexpr (W > 1) {
                if (lane == 0) sh.any[wave] = alive;
                __syncthreads();  // (and the waves are done with the previous batch)
                uint32_t any = 0;
#pragma unroll
                for (int w = 0; w < W; ++w) any |= sh.any[w];
                if (!any) break;
            } else {
                if (!alive) break;
            }
        }
        stage_batch(sh, vt, c, b0, rg.y, pval, rec, ioff);
        staged = b0;
        __syncthreads();
        for (int s = 0; s < W && alive && b0 + (uint32_t)(s * kWave) < rg.y; ++s) {
            const uint32_t mask = __float_as_uint(sh.d[s * kWave + lane].y) >> (wave * RPL);
#pragma unroll
            for (int k = 0; k < RPL; k += KP) {
                if (!(alive >> (k / KP) & 1u)) continue;
                const unsigned long long m = __ballot((mask >> k & ((1u << KP) - 1u)) != 0u);
                if (!forward_list<KP, W, STATS>(sh, m, s, b0 - rg.x, pxl, pyl + (float)(4 * k), T + k, C0 + k, C1 + k,
                                                C2 + k, last + k, ncontrib + k, stop_at + k))
                    alive &= ~(1u << (k / KP));
            }
        }
    }
}

// Lanes [0, 32) of the result: x of the lane and of the lane 32 above, added;
// lanes [32, 64): the same of y.
__device__ __forceinline__ float swap_add32(float x, float y) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// Rows of 16 lanes of the result: x rows 0 + 1, y rows 0 + 1, x rows 2 + 3, y rows 2 + 3.
__device__ __forceinline__ float swap_add16(float x, float y) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// x y, and 0 where either is 0, whatever the other (v_mul_legacy_f32; as the
// compiler's intrinsic, so that it keeps the waits before the lane swaps that
// read the product).
__device__ float mul_legacy(float x, float y) __asm("llvm.amdgcn.fmul.legacy");

// A record's part of the lanes of `on` and of no others: with w = alpha T, the
// colour gradient sums (zero before the first of RPL rows), gB (g . the colour
// behind the record, grgb = g . its own) and T.  w is undefined elsewhere.  By
// the execution mask, which costs no vector instruction where selects would; but a
// wave of one slab is one of few, and waits for its chain through T and gB, which
// the mask's changes lengthen (71.8 against 70.5 us at 128 x 128), so there by
// selects, and by the product that is 0 where w is, whatever the other factor.
template <int RPL>
__device__ __forceinline__ void backward_add(unsigned long long on, float alpha, float g0, float g1, float g2,
                                             float grgb, float &a_c0, float &a_c1, float &a_c2, float &gB, float &T,
                                             float &w) {
    if constexpr (RPL == 1) {
        const bool ok = __builtin_amdgcn_inverse_ballot_w64(on);
        w = ok ? alpha * T : 0.f;
        a_c0 = mul_legacy(w, g0);
        a_c1 = mul_legacy(w, g1);
        a_c2 = mul_legacy(w, g2);
        gB = ok ? fmaf(-w, grgb, gB) : gB;
        T -= w;  // T (1 - alpha)
    } else {
        unsigned long long all;
        asm("s_and_saveexec_b64 %[all], %[on]\n\t"
            "v_mul_f32 %[w], %[alpha], %[T]\n\t"
            "v_fmac_f32 %[a_c0], %[w], %[g0]\n\t"
            "v_fmac_f32 %[a_c1], %[w], %[g1]\n\t"
            "v_fmac_f32 %[a_c2], %[w], %[g2]\n\t"
            "v_fma_f32 %[gB], -%[w], %[grgb], %[gB]\n\t"
            "v_sub_f32 %[T], %[T], %[w]\n\t"
            "s_mov_b64 exec, %[all]"
            : [all] "=&s"(all), [w] "=&v"(w), [a_c0] "+v"(a_c0), [a_c1] "+v"(a_c1), [a_c2] "+v"(a_c2), [gB] "+v"(gB),
              [T] "+v"(T)
            : [on] "s"(on), [alpha] "v"(alpha), [g0] "v"(g0), [g1] "v"(g1), [g2] "v"(g2), [grgb] "v"(grgb)
            : "scc");
    }
}

// A7 for one tile over list positions [rg.x, end); `staged`: the position of
// the batch the forward left staged (a fused step's), or anything but rg.x for
// none.  The per-pixel state starts at T = 1, g = dL/dC, gB = g . C_out and the
// contributor count ncon.
template <int RPL, int W>
__device__ __forceinline__ void tile_backward(Staged<W> &sh, Reduce<W> &bw, const ViewTable &vt, const TileCtx &c,
                                              uint2 rg, uint32_t end, uint32_t staged,
                                              const uint32_t *__restrict__ pval, const Rec *__restrict__ rec,
                                              const uint32_t *__restrict__ ioff, int wave, int lane, float pxl, float pyl,
                                              float (&T)[RPL], const float (&g0)[RPL], const float (&g1)[RPL],
                                              const float (&g2)[RPL], float (&gB)[RPL], const uint32_t (&ncon)[RPL],
                                              float *__restrict__ partial, uint8_t *__restrict__ pflag) {
    const uint32_t tid = threadIdx.x;
    uint32_t mine = 0;
#pragma unroll
    for (int k = 0; k < RPL; ++k) mine = max(mine, ncon[k]);
    // positions this wave's pixels used end here
    const uint32_t stop = rg.x + wave_reduce(mine, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
    // the (Gaussian of the group, moment) this lane finalises
    const int fq = lane / kPartialStride, fc = lane - fq * kPartialStride;
    float *red = bw.red[wave];
    for (uint32_t b0 = rg.x; b0 < end; b0 += W * kWave) {
        if (b0 != rg.x || staged != rg.x) {  // (the forward's batch is there only if it is the first)
            if (b0 != rg.x) __syncthreads();
            stage_batch(sh, vt, c, b0, end, pval, rec, ioff);
            if (b0 == rg.x) stage_sentinel(sh);
            __syncthreads();
        }
        for (int s = 0; s < W; ++s) {
            const uint32_t s0 = b0 + (uint32_t)(s * kWave);
            if (s0 >= end) break;
            unsigned long long m = 0ull;
            if (s0 < stop) {
                const uint32_t mask = __float_as_uint(sh.d[s * kWave + lane].y) >> (wave * RPL);
                m = __ballot((mask & ((1u << RPL) - 1u)) != 0u);
                if (stop - s0 < (uint32_t)kWave) m &= (1ull << (stop - s0)) - 1ull;
            }
            if constexpr (W > 1)
                if (lane == 0) bw.live[wave] = m;
            while (m) {
                int j[kGroup];
                uint32_t packed;
                const int n = take_group<W>(m, s, j, packed);
                // per lane: the sums over its rows of sa = alpha dL/dalpha, sa dy,
                // sa dy^2 and the colour gradient (the rows share dx)
                float v[kGroup][6];
#pragma unroll
                for (int q = 0; q < kGroup; ++q) {
                    const float4 a = sh.a[j[q]], b = sh.b[j[q]];
                    const float2 d = *reinterpret_cast<const float2 *>(&sh.d[j[q]]);
                    const float dx = a.x - pxl;
                    const uint32_t pos = b0 - rg.x + (uint32_t)j[q];
                    const RowQuad rq = row_quad(a, b, dx);
                    const uint32_t smask = RPL > 1 ? slab_mask(d.y) >> (wave * RPL) : 1u;
                    float a_c0 = 0.f, a_c1 = 0.f, a_c2 = 0.f, a_sa = 0.f, a_say = 0.f, a_sayy = 0.f;
#pragma unroll
                    for (int k = 0; k < RPL; ++k) {
                        if (RPL > 1 && !(smask & (1u << k))) continue;
                        const float dy = a.y - (pyl + (float)(4 * k));
                        const float araw = raw_alpha(alpha_exponent(rq, b, dy));
                        const float alpha = fminf(kAlphaMax, araw);
                        const unsigned long long on = __ballot(pos < ncon[k]) & __ballot(alpha >= kAlphaMin);
                        const float grgb = fmaf(g0[k], b.z, fmaf(g1[k], b.w, g2[k] * d.x));
                        // alpha dL/dalpha = alpha T g.c - alpha g.B / (1 - alpha), with
                        // B the colour behind this Gaussian; with w = alpha T and
                        // T' = T (1 - alpha) that is w (g.c - g.B / T')
                        float w;
                        backward_add<RPL>(on, alpha, g0[k], g1[k], g2[k], grgb, a_c0, a_c1, a_c2, gB[k], T[k], w);
                        const float h = fmaf(-gB[k], __builtin_amdgcn_rcpf(T[k]), grgb);
                        // dL/dsigma = -sa, alpha dL/dalpha = sa (zero where the Gaussian
                        // adds nothing and through the 0.99 clamp)
                        const float sa_ =
                            __builtin_amdgcn_inverse_ballot_w64(on & __ballot(araw < kAlphaMax)) ? w * h : 0.f;
                        a_sa += sa_;
                        const float say = sa_ * dy;
                        a_say += say;
                        a_sayy = fmaf(say, dy, a_sayy);
                    }
                    v[q][0] = a_sa, v[q][1] = a_say, v[q][2] = a_sayy;
                    v[q][3] = a_c0, v[q][4] = a_c1, v[q][5] = a_c2;
                }
                // sums over the wave's four rows of 16 lanes; row q of the result holds Gaussian q's
                float r[6];
#pragma unroll
                for (int cc = 0; cc < 6; ++cc)
                    r[cc] = swap_add16(swap_add32(v[0][cc], v[2][cc]), swap_add32(v[1][cc], v[3][cc]));
                const float dxr = sh.a[s * kWave + (int)(packed >> (8 * (lane >> 4)) & 63u)].x - pxl;
                // the moments of sa (= -dL/dsigma): sums of sa dx, sa dy, sa dx^2,
                // sa dx dy, sa dy^2 (the negated S_x .. S_yy of the projection
                // backward), then S_o = sum sa and the colour gradient
                const float sx = dxr * r[0];
                red[0 * kRedStride + lane] = sx;
                red[1 * kRedStride + lane] = r[1];
                red[2 * kRedStride + lane] = dxr * sx;
                red[3 * kRedStride + lane] = dxr * r[1];
                red[4 * kRedStride + lane] = r[2];
                red[5 * kRedStride + lane] = r[0];
                red[6 * kRedStride + lane] = r[3];
                red[7 * kRedStride + lane] = r[4];
                red[8 * kRedStride + lane] = r[5];
                // (the wave's own LDS accesses, in order: no barrier, only no reordering by the compiler)
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                if (fq < n) {
                    const float4 *rr = reinterpret_cast<const float4 *>(red + fc * kRedStride + fq * 16);
                    const float4 x = rr[0], y = rr[1], z = rr[2], w = rr[3];
                    const float t = (((x.x + x.y) + (x.z + x.w)) + ((y.x + y.y) + (y.z + y.w))) +
                                    (((z.x + z.y) + (z.z + z.w)) + ((w.x + w.y) + (w.z + w.w)));
                    const uint32_t jl = packed >> (8 * fq) & 63u;
                    if constexpr (W > 1) {
                        bw.mom[wave][jl * kPartialStride + fc] = t;
                    } else {
                        const uint32_t p = __float_as_uint(sh.d[jl].z);
                        partial[(size_t)p * kPartialStride + fc] = t;
                        if (fc == 0) pflag[p] = 1;  // this pair has moments: the reduction reads them
                    }
                }
            }
            if constexpr (W > 1) {
                __syncthreads();
                const uint32_t vals = min((uint32_t)kWave, end - s0) * kPartialStride;
                for (uint32_t e = tid; e < vals; e += W * kWave) {
                    const uint32_t jj = e / kPartialStride, cc = e - jj * kPartialStride;
                    float t = 0.f;
                    bool any = false;
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        const bool on = (bw.live[w] >> jj) & 1ull;
                        t += on ? bw.mom[w][e] : 0.f;
                        any |= on;
                    }
                    if (any) {
                        const uint32_t p = __float_as_uint(sh.d[s * kWave + jj].z);
                        partial[(size_t)p * kPartialStride + cc] = t;
                        if (cc == 0) pflag[p] = 1;
                    }
                }
                __syncthreads();
            }
        }
    }
}

// Tile turn of the workgroup (all its waves get it).
template <int W>
__device__ __forceinline__ uint32_t next_turn(bool persistent, uint32_t *queue, uint32_t &iter, uint32_t *s_turn) {
    if (!persistent) return iter++ == 0 ? blockIdx.x : 0xffffffffu;
    __syncthreads();
    if (threadIdx.x == 0) *s_turn = atomicAdd(queue, 1u);
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*s_turn);
}

// Largest of the workgroup's values.
template <int W>
__device__ __forceinline__ uint32_t group_max(uint32_t v, uint32_t *s /* [W] */) {
    v = wave_reduce(v, 0u, [](uint32_t a, uint32_t b) { return max(a, b); });
    if constexpr (W == 1) return v;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) s[threadIdx.x >> 6] = v;
    __syncthreads();
    uint32_t r = 0;
#pragma unroll
    for (int w = 0; w < W; ++w) r = max(r, s[w]);
    return __builtin_amdgcn_readfirstlane(r);
}

// One kernel body for the three passes: forward only, backward only (from the
// state a forward left), or the fused step.
struct CompositeArgs {
    const uint2 *ranges;
    const uint32_t *pval;
    const Rec *rec;
    const uint32_t *ioff;  // pair offsets, for the backward's moments
    float3 bg;
    Upstream up;
    float *out_rgb, *out_T, *pix_T;
    uint32_t *pix_n, *tile_cut, *tile_order;
    float *partial;
    uint8_t *pflag;
    ZeroRows zr;
    WsHeader *hdr;
    int persistent;
};

template <int RPL, int W, bool FWD, bool BWD, bool STATS>
__global__ __launch_bounds__(W *kWave) void k_composite(ViewTable vt, CompositeArgs A) {
    __shared__ Staged<W> sh;
    __shared__ uint32_t s_turn;
    const int lane = threadIdx.x & 63, wave = W > 1 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int lx = lane & 15, ly = wave * 4 * RPL + (lane >> 4);
    const float pxl = (float)lx + 0.5f, pyl = (float)ly + 0.5f;
    uint32_t iter = 0;
    for (;;) {
        const uint32_t r = next_turn<W>(A.persistent != 0, &A.hdr->queue[FWD ? 0 : 1], iter, &s_turn);
        if (r >= vt.total_tiles) break;
        // (the tile is one for the wave: scalar registers and loads from here on)
        const uint32_t t = __builtin_amdgcn_readfirstlane(BWD ? tile_by_cost(A.tile_order, vt.total_tiles, r) : r);
        if constexpr (BWD) zero_unseen_rows(A.zr, t, A.hdr->overflow != 0u, (int)threadIdx.x, W * kWave);
        const TileCtx c = tile_ctx(vt, t);
        const uint2 rg = A.ranges[t];
        const uint32_t infinite = FWD ? __builtin_amdgcn_readfirstlane(A.hdr->infinite) : 0u;  // (asked for early)
        const uint32_t px = c.ox + lx;
        const size_t plane = (size_t)c.width * c.height;
        float *img = A.out_rgb + 3 * (size_t)c.pix_off;
        float T[RPL], C0[RPL], C1[RPL], C2[RPL];
        uint32_t last[RPL], stop_at[RPL], ncontrib[RPL], staged = 0xffffffffu, nmax = 0;
        if constexpr (FWD) {
#pragma unroll
            for (int k = 0; k < RPL; ++k) {
                const uint32_t py = c.oy + ly + 4 * k;
                T[k] = (px < c.width && py < c.height) ? 1.f : -1.f;
                C0[k] = C1[k] = C2[k] = 0.f;
                last[k] = 0;
                ncontrib[k] = 0;
                stop_at[k] = 0xffffffffu;
            }
            tile_forward<RPL, W, forward_slabs(RPL), STATS>(sh, vt, c, rg, A.pval, A.rec, BWD ? A.ioff : nullptr, wave, lane, pxl, pyl, T, C0, C1, C2,
                                           last, ncontrib, stop_at, staged);
        }
        // the forward's outputs, and the backward's start: g = dL/dC, gB = g . C_out
        // (gB: g . the colour still to come behind the current position)
        const float *gimg = (A.up.target ? A.up.target : A.up.grad) + 3 * (size_t)c.pix_off;
        float g0[RPL], g1[RPL], g2[RPL], gB[RPL];
        uint32_t evals = 0, replays = 0, contrib = 0;
#pragma unroll
        for (int k = 0; k < RPL; ++k) {
            const uint32_t py = c.oy + ly + 4 * k;
            g0[k] = g1[k] = g2[k] = gB[k] = 0.f;
            if (px < c.width && py < c.height) {
                const size_t pix = (size_t)py * c.width + px;
                float i0, i1, i2;
                if constexpr (FWD) {
                    const float Tf = fabsf(T[k]);
                    i0 = C0[k] + Tf * A.bg.x, i1 = C1[k] + Tf * A.bg.y, i2 = C2[k] + Tf * A.bg.z;
                    if (infinite) {  // uniform (the products are infinite)
                        i0 = C0[k] < kColourInfinite ? i0 : C0[k] * kColourInfinite;
                        i1 = C1[k] < kColourInfinite ? i1 : C1[k] * kColourInfinite;
                        i2 = C2[k] < kColourInfinite ? i2 : C2[k] * kColourInfinite;
                    }
                    img[pix] = i0;
                    img[plane + pix] = i1;
                    img[2 * plane + pix] = i2;
                    A.pix_T[c.pix_off + pix] = Tf;
                    A.pix_n[c.pix_off + pix] = last[k];
                    if (A.out_T) A.out_T[c.pix_off + pix] = Tf;
                    nmax = max(nmax, last[k]);
                    if constexpr (STATS) {
                        evals += stop_at[k] != 0xffffffffu ? stop_at[k] + 1 : rg.y - rg.x;
                        replays += last[k];
                        contrib += ncontrib[k];
                    }
                } else {
                    last[k] = A.pix_n[c.pix_off + pix];
                    i0 = img[pix], i1 = img[plane + pix], i2 = img[2 * plane + pix];
                }
                if constexpr (BWD) {
                    g0[k] = gimg[pix];
                    g1[k] = gimg[plane + pix];
                    g2[k] = gimg[2 * plane + pix];
                    if (A.up.target) {  // mean absolute error: dL/dC = sign(C - target) / count
                        g0[k] = l1_grad(i0, g0[k], A.up.l1_scale);
                        g1[k] = l1_grad(i1, g1[k], A.up.l1_scale);
                        g2[k] = l1_grad(i2, g2[k], A.up.l1_scale);
                    }
                    gB[k] = fmaf(g2[k], i2, fmaf(g1[k], i1, g0[k] * i0));
                }
            } else {
                last[k] = 0;
            }
            T[k] = 1.f;
        }
        if constexpr (STATS) {
            // work counters for the measurement harness (integer adds: order independent)
            unsigned long long e = evals, rp = replays, cc = contrib;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) {
                e += __shfl_xor(e, o, kWave);
                rp += __shfl_xor(rp, o, kWave);
                cc += __shfl_xor(cc, o, kWave);
            }
            if (lane == 0) {
                atomicAdd(&A.hdr->evaluations, e);
                atomicAdd(&A.hdr->replays, rp);
                atomicAdd(&A.hdr->contributors, cc);
            }
        }
        if constexpr (FWD) {
            nmax = group_max<W>(nmax, sh.any);
            if (threadIdx.x == 0) {
                A.tile_cut[t] = nmax;  // positions the backward replays
                if constexpr (!BWD) {  // the backward's schedule: this tile in the bucket of its replay count
                    const uint32_t b = cost_bucket(nmax);
                    const uint32_t slot = atomicAdd(&A.tile_order[b], 1u);
                    A.tile_order[kCostBuckets + (size_t)b * vt.total_tiles + slot] = t;
                }
            }
        } else {
            nmax = A.tile_cut[t];
        }
        if constexpr (BWD) {
            __shared__ Reduce<W> bw;
            tile_backward<RPL, W>(sh, bw, vt, c, rg, rg.x + nmax, staged, A.pval, A.rec, A.ioff, wave, lane, pxl, pyl, T,
                                  g0, g1, g2, gB, last, A.partial, A.pflag);
        }
    }
}

// Waves per tile.  The forward takes as many as it can (16 x 16 tiles, W = 1 / 2 /
// 4: 136 / 95 / 74 us at 1,200 tiles, 151 / 151 / 142 us at 8,160; 16 x 8 tiles, W = 1 /
// 2: 197 / 184 us at 16,200) but where the tiles alone fill the chip many times over:
// there, what each wave repeats counts for more.  Whole forwards, us, of 300 k
// Gaussians evenly spread, 1.5 M, and 300 k in the middle, whose longest lists take
// most of the time: 16 x 16, W = 1 / 4: 302 / 288, 504 / 508 and 779 / 632 at 14,400
// tiles, 471 / 508, 852 / 917 and 5,324 / 5,135 at 32,400, 1,377 / 1,631, 2,985 / 3,345
// and 16,877 / 16,865 at 129,600; 16 x 32, W = 2 / 4: 434 / 439, 707 / 728 and 773 / 696
// at 16,200, 1,225 / 1,343, 2,137 / 2,316 and 9,303 / 9,324 at 64,800; 16 x 8, W = 1 / 2: no
// difference.  The line is where no scene loses.
static int forward_waves(const ViewTable &vt) {
    if (vt.tile_h >= 16 && vt.total_tiles > 40000u) return vt.tile_h == 16 ? 1 : 2;
    return vt.tile_h / 4 < 4 ? vt.tile_h / 4 : 4;
}

// The backward and the fused step (one rule: both must add up a pair's moments
// in the same order) give a wave fewer slabs the fewer tiles there are.
// Measured on the fused step with 400k Gaussians at two distances (dense and
// even; concentrated in the centre), us:
//   1 slab per wave against one wave per tile   16 x 16: 214 / 369 and 371 / 901
//     at 1,200 tiles, 229 / 246 and 355 / 533 at 2,952, 255 / 241 and 365 /
//     512 at 3,600; 16 x 8: 201 / 231 and 343 / 475 at 2,400, 211 / 201 and
//     320 / 418 at 3,750, 241 / 200 and 327 / 342 at 5,832
//   2 slabs against one wave   16 x 16: 253 / 241 and 409 / 512 at 3,600, 319 /
//     272 and 422 / 452 at 5,700; 16 x 32: 381 / 384 and 470 / 649 at 4,080
//   4 slabs against one wave   16 x 32: 851 / 893 and 1266 / 1305 at 7,360, but
//     1235 / 1178 at 14,720 (even)
static int backward_waves(const ViewTable &vt) {
    const int slabs = vt.tile_h / 4;
    const uint32_t tiles = vt.total_tiles;
    const int per_wave = tiles <= 3200u ? 1 : tiles <= 4500u ? 2 : tiles <= 9000u ? 4 : 8;
    const int waves = slabs <= per_wave ? 1 : slabs / per_wave;
    return waves < 4 ? waves : 4;
}

// Workgroups of a persistent launch: as many as can be resident at once
// (occupancy of this kernel x compute units of the current device, queried at
// each launch: nothing is cached between calls), unless the caller fixed it.
template <typename Kernel>
static int resident_ctas(Kernel kernel, int requested, int threads = kWave) {
    if (requested > 0) return requested;
    int dev = 0, cus = 0, per = 0;
    if (hipGetDevice(&dev) != hipSuccess) dev = 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) cus = 256;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kernel, threads, 0) != hipSuccess || per <= 0) per = 8;
    return cus * per;
}

// One pass over the tiles in the form the call takes.
template <bool FWD, bool BWD, bool STATS>
static void launch_composite(const ViewTable &vt, const CompositeArgs &A, int persistent_ctas, hipStream_t st) {
#define GSR_COMPOSITE(R, W)                                                                                         \
    hipLaunchKernelGGL((k_composite<R, W, FWD, BWD, STATS>),                                                        \
                       dim3(A.persistent ? (unsigned)resident_ctas(k_composite<R, W, FWD, BWD, STATS>,              \
                                                                   persistent_ctas, W * kWave)                      \
                                         : vt.total_tiles),                                                         \
                       dim3(W * kWave), 0, st, vt, A)
    const int waves = BWD ? backward_waves(vt) : forward_waves(vt);
    if (waves == 1 && vt.tile_h == 16) {
        GSR_COMPOSITE(4, 1);
        return;
    }
    if (waves == 2 && vt.tile_h == 32) {
        GSR_COMPOSITE(4, 2);
        return;
    }
    if constexpr (BWD) {  // (forms the forward alone does not take)
        if (waves == 1 && vt.tile_h > 4) {
            if (vt.tile_h == 8) GSR_COMPOSITE(2, 1);
            else GSR_COMPOSITE(8, 1);
            return;
        }
        if (waves == 2 && vt.tile_h == 16) {
            GSR_COMPOSITE(2, 2);
            return;
        }
    }
    switch (vt.tile_h) {
        case 4: GSR_COMPOSITE(1, 1); break;
        case 8: GSR_COMPOSITE(1, 2); break;
        case 32: GSR_COMPOSITE(2, 4); break;
        default: GSR_COMPOSITE(1, 4); break;
    }
#undef GSR_COMPOSITE
}

void launch_composite_fwd(const ViewTable &vt, const uint2 *ranges, const uint32_t *pval, const Rec *rec,
                          float3 bg, float *out_rgb, float *out_T, float *pix_T,
                          uint32_t *pix_n, uint32_t *tile_cut, uint32_t *tile_order, WsHeader *hdr,
                          bool persistent, int persistent_ctas, bool stats, hipStream_t st) {
    if (vt.total_tiles == 0) return;
    CompositeArgs A{};
    A.ranges = ranges, A.pval = pval, A.rec = rec, A.bg = bg;
    A.out_rgb = out_rgb, A.out_T = out_T, A.pix_T = pix_T, A.pix_n = pix_n;
    A.tile_cut = tile_cut, A.tile_order = tile_order, A.hdr = hdr, A.persistent = persistent ? 1 : 0;
    if (stats) launch_composite<true, false, true>(vt, A, persistent_ctas, st);
    else launch_composite<true, false, false>(vt, A, persistent_ctas, st);
}

void launch_composite_bwd(const ViewTable &vt, const uint2 *ranges, const uint32_t *pval, const Rec *rec,
                          const uint32_t *ioff, const float *out_rgb, const Upstream &up, const uint32_t *pix_n,
                          const uint32_t *tile_cut, const uint32_t *tile_order, float *partial, uint8_t *pflag,
                          const ZeroRows &zr, WsHeader *hdr, bool persistent, int persistent_ctas, hipStream_t st) {
    if (vt.total_tiles == 0) return;
    CompositeArgs A{};
    A.ranges = ranges, A.pval = pval, A.rec = rec, A.ioff = ioff, A.up = up;
    A.out_rgb = const_cast<float *>(out_rgb), A.pix_n = const_cast<uint32_t *>(pix_n);
    A.tile_cut = const_cast<uint32_t *>(tile_cut), A.tile_order = const_cast<uint32_t *>(tile_order);
    A.partial = partial, A.pflag = pflag, A.zr = zr, A.hdr = hdr, A.persistent = persistent ? 1 : 0;
    launch_composite<false, true, false>(vt, A, persistent_ctas, st);
}

void launch_composite_step(const ViewTable &vt, const uint2 *ranges, const uint32_t *pval, const Rec *rec,
                           const uint32_t *ioff, float3 bg, const float *target, float l1_scale, float *out_rgb,
                           float *out_T, float *pix_T, uint32_t *pix_n, uint32_t *tile_cut,
                           const uint32_t *tile_order, float *partial, uint8_t *pflag, const ZeroRows &zr,
                           WsHeader *hdr, bool persistent, int persistent_ctas, hipStream_t st) {
    if (vt.total_tiles == 0) return;
    CompositeArgs A{};
    A.ranges = ranges, A.pval = pval, A.rec = rec, A.ioff = ioff, A.bg = bg, A.up = Upstream{nullptr, target, l1_scale};
    A.out_rgb = out_rgb, A.out_T = out_T, A.pix_T = pix_T, A.pix_n = pix_n;
    A.tile_cut = tile_cut, A.tile_order = const_cast<uint32_t *>(tile_order);
    A.partial = partial, A.pflag = pflag, A.zr = zr, A.hdr = hdr, A.persistent = persistent ? 1 : 0;
    launch_composite<true, true, false>(vt, A, persistent_ctas, st);
}

}  // namespace gsr
