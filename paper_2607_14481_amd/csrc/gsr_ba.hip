// gsr_ba.hip -- local bundle adjustment with a dense Schur complement on
// gfx950, in FP64 (Sec. 5.1, "Local Bundle Adjustment" and "Solver
// efficiency"; appendix "Details on Local Pose Reconstruction", paragraph
// "Fast Bundle Adjustment").
//
// Unknowns: the free keyframe poses (a left twist (rho, phi) each, translation
// first), one shared focal length f, and the landmarks.  Residual of the
// observation of landmark j in keyframe i: f (X / Z, Y / Z) + c - z_ij with
// X = R_i p_j + t_i.  One iteration is a Levenberg-Marquardt step with
// Marquardt damping (every diagonal of the normal matrix scaled by 1 + lambda)
// taken unconditionally:
//
//   k_ba_landmark   one 8-lane group per landmark, one lane per observation
//                   slot: takes the previous step's landmark update (back-
//                   substitution at the previous linearisation point), then
//                   residual and Jacobians at the new one and the landmark's
//                   3x3 block (damped, inverted in closed form); writes one
//                   128-byte record per landmark;
//   k_ba_assemble   workgroups per block (a, b) of the reduced camera
//                   system, each walking its part of a host-built list of
//                   the landmarks the two keyframes share in a fixed order
//                   (deterministic, no atomics) into a partial system, plus
//                   workgroups for the focal-length entry and the cost;
//   k_ba_solve      one workgroup: adds the partial systems, a blocked
//                   L D L^T on the FP64 matrix cores, the two triangular
//                   solves, the SE(3) retraction of the free poses and the
//                   focal step.
//
// Nothing is stored per observation.  With H^-1 the inverse of the damped
// landmark block, a pair of observations o (keyframe a) and q (keyframe b) of
// one landmark contributes
//   Jx_o^T M Jx_q,  M = -Jp_o H^-1 Jp_q^T  (2 x 2)
// to block (a, b), and an observation to the diagonal block, the focal column
// and the right-hand side
//   Jx^T (I - Jp H^-1 Jp^T) Jx,  Jx^T (Jf - Jp H^-1 b_f),  Jx^T (r - Jp H^-1 g_p)
// (b_f = sum over the landmark's observations of Jf^T Jp, g_p the landmark
// gradient; the damping lambda diag(Jx^T Jx) is added per block).  The
// assembly evaluates the Jacobians again from the landmark's record (its
// position, H^-1, b_f, g_p: one cache line) and the block's two poses, which
// the whole workgroup shares: about 200 FP64 operations per pair instead of
// reading 288 bytes of stored factors.  At 20 keyframes x 10,000 landmarks
// (49,891 observations) an iteration so moves about 10 MB instead of 69 MB;
// with 24 MB less to write, the landmark pass (the update included) takes 6.2
// instead of 16 + 5 us and the assembly 12.3 instead of 19.6 us.
#include "gsr_ba.h"

namespace gsr {

namespace {

constexpr int kLanesPerLm = kBaMaxObs;   // 8
constexpr int kBaThreads = 256;
constexpr int kLmPerBlock = kBaThreads / kLanesPerLm;
constexpr int kAsmThreads = 512;
constexpr int kSolveThreads = 1024;
constexpr int kTile = 16;                // rows and columns of a matrix-core tile
constexpr int kMaxTiles = (6 * kBaMaxFree + 2 + kTile - 1) / kTile;   // 8: tile rows of the largest system

// offsets inside a landmark record: position, inverse block (00 01 02 11 12 22), b_f, g_p
constexpr int kQP = 0, kQH = 3, kQB = 9, kQG = 12;

// One DPP step on a double (both 32-bit halves moved alike): v + v moved
// across lanes by `ctrl`, only in the rows enabled by `row_mask` (others add 0).
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add_d(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    int lo = (int)(unsigned)b, hi = (int)(unsigned)(b >> 32);
    if constexpr (ROW_MASK == 0xf) {
        lo = __builtin_amdgcn_mov_dpp(lo, CTRL, 0xf, 0xf, true);
        hi = __builtin_amdgcn_mov_dpp(hi, CTRL, 0xf, 0xf, true);
    } else {
        lo = __builtin_amdgcn_update_dpp(0, lo, CTRL, ROW_MASK, 0xf, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, CTRL, ROW_MASK, 0xf, false);
    }
    return v + __longlong_as_double((long long)(((unsigned long long)(unsigned)hi << 32) | (unsigned)lo));
}

__device__ __forceinline__ double readlane_d(double v, int l) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// Sum over an 8-lane group (one landmark's observation slots): two quad swaps
// give each lane its quad's sum, the half-row mirror adds the other quad's.
// Additions pair the same operands on every lane, so all 8 lanes hold the
// bit-identical total.
__device__ __forceinline__ double group_sum(double v) {
    v = dpp_add_d<0xB1, 0xf>(v);   // quad_perm [1, 0, 3, 2]
    v = dpp_add_d<0x4E, 0xf>(v);   // quad_perm [2, 3, 0, 1]
    return dpp_add_d<0x141, 0xf>(v);  // row_half_mirror
}

// Lane swaps of a double (both halves): swap32(x, y)'s lanes [0, 32) hold x
// of the lane plus x of the lane 32 above, lanes [32, 64) the same of y;
// swap16's rows of 16 lanes hold x rows 0 + 1, y rows 0 + 1, x rows 2 + 3,
// y rows 2 + 3.
struct Halves {
    unsigned lo, hi;
};
__device__ __forceinline__ Halves halves(double v) {
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    return Halves{(unsigned)b, (unsigned)(b >> 32)};
}
__device__ __forceinline__ double whole(unsigned lo, unsigned hi) {
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ double swap_add32_d(double x, double y) {
    const Halves a = halves(x), b = halves(y);
    const auto l = __builtin_amdgcn_permlane32_swap(a.lo, b.lo, false, false);
    const auto h = __builtin_amdgcn_permlane32_swap(a.hi, b.hi, false, false);
    return whole(l[0], h[0]) + whole(l[1], h[1]);
}
__device__ __forceinline__ double swap_add16_d(double x, double y) {
    const Halves a = halves(x), b = halves(y);
    const auto l = __builtin_amdgcn_permlane16_swap(a.lo, b.lo, false, false);
    const auto h = __builtin_amdgcn_permlane16_swap(a.hi, b.hi, false, false);
    return whole(l[0], h[0]) + whole(l[1], h[1]);
}

// Sum of N per-thread accumulators over a block of WAVES waves in a fixed
// order (deterministic).  Four values at a time: two lane-swap levels leave
// one register whose rows of 16 lanes hold values 0, 2, 1 and 3, four DPP
// steps add each row (5 cross-lane steps per value instead of 18); then
// thread t adds the waves' value t in wave order.  red: WAVES + 1 times (N
// rounded up to 4) doubles of LDS; returns the N sums (in LDS, valid for every thread).
template <int WAVES, int N>
__device__ __forceinline__ const double *block_sum(const double (&acc)[N], double *red) {
    constexpr int R = (N + 3) / 4 * 4;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int row = lane >> 4, pick = row == 1 ? 2 : (row == 2 ? 1 : row);
#pragma unroll
    for (int t = 0; t < R; t += 4) {
        const double v0 = acc[t], v1 = t + 1 < N ? acc[t + 1 < N ? t + 1 : 0] : 0.0;
        const double v2 = t + 2 < N ? acc[t + 2 < N ? t + 2 : 0] : 0.0, v3 = t + 3 < N ? acc[t + 3 < N ? t + 3 : 0] : 0.0;
        double v = swap_add16_d(swap_add32_d(v0, v1), swap_add32_d(v2, v3));
        v = dpp_add_d<0xB1, 0xf>(v);   // quad_perm [1, 0, 3, 2]
        v = dpp_add_d<0x4E, 0xf>(v);   // quad_perm [2, 3, 0, 1]
        v = dpp_add_d<0x141, 0xf>(v);  // row_half_mirror
        v = dpp_add_d<0x140, 0xf>(v);  // row_mirror
        if ((lane & 15) == 0) red[w * R + t + pick] = v;
    }
    __syncthreads();
    if (threadIdx.x < N) {
        const int t = threadIdx.x;
        double v = red[t];
#pragma unroll
        for (int q = 1; q < WAVES; ++q) v += red[q * R + t];
        red[WAVES * R + t] = v;
    }
    __syncthreads();
    return red + WAVES * R;
}

// A partial system: D rows of pitch D + 1 (even, as D = 6F + 1 is odd, so rows
// are 16-byte aligned), then the right-hand side (D), the cost and a pad.
__device__ __forceinline__ size_t part_stride(int D) { return (size_t)(D + 1) * (D + 1); }

// Camera-frame point of an observation and the derivatives of its projection:
// d pi / dX = [[a, 0, b], [0, a, c]].
struct ObsGeom {
    double x, y, z, xn, yn, a, b, c;
};

__device__ __forceinline__ ObsGeom observe(const double *__restrict__ T, const double p[3], double f) {
    ObsGeom o;
    o.x = fma(T[0], p[0], fma(T[1], p[1], fma(T[2], p[2], T[3])));
    o.y = fma(T[4], p[0], fma(T[5], p[1], fma(T[6], p[2], T[7])));
    o.z = fma(T[8], p[0], fma(T[9], p[1], fma(T[10], p[2], T[11])));
    const double iz = 1.0 / o.z;
    o.xn = o.x * iz;
    o.yn = o.y * iz;
    o.a = f * iz;
    o.b = -o.a * o.xn;
    o.c = -o.a * o.yn;
    return o;
}

// Jacobian rows with respect to the pose's left twist: dX/drho = I, dX/dphi = -[X]x.
__device__ __forceinline__ void pose_rows(const ObsGeom &o, double (&j0)[6], double (&j1)[6]) {
    j0[0] = o.a;  j0[1] = 0.0;  j0[2] = o.b;
    j0[3] = o.b * o.y;  j0[4] = o.a * o.z - o.b * o.x;  j0[5] = -o.a * o.y;
    j1[0] = 0.0;  j1[1] = o.a;  j1[2] = o.c;
    j1[3] = o.c * o.y - o.a * o.z;  j1[4] = -o.c * o.x;  j1[5] = o.a * o.x;
}

// Jacobian rows with respect to the landmark.
__device__ __forceinline__ void point_rows(const ObsGeom &o, const double *__restrict__ T, double (&j0)[3], double (&j1)[3]) {
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        j0[k] = fma(o.a, T[k], o.b * T[8 + k]);
        j1[k] = fma(o.a, T[4 + k], o.c * T[8 + k]);
    }
}

// h (packed symmetric 3x3) times v
__device__ __forceinline__ void sym3(const double *h, const double v[3], double (&o)[3]) {
    o[0] = fma(h[0], v[0], fma(h[1], v[1], h[2] * v[2]));
    o[1] = fma(h[1], v[0], fma(h[3], v[1], h[4] * v[2]));
    o[2] = fma(h[2], v[0], fma(h[4], v[1], h[5] * v[2]));
}

__device__ __forceinline__ double dot3(const double a[3], const double b[3]) {
    return fma(a[0], b[0], fma(a[1], b[1], a[2] * b[2]));
}

// flags: kUpdate: first take the landmark update of the step the solve has
// just finished; kCostOnly: nothing but the cost after that.
constexpr int kUpdate = 1, kCostOnly = 2;

__global__ void __launch_bounds__(kBaThreads) k_ba_landmark(BaArgs A, int flags) {
    __shared__ double red[5 * 4];
    const uint32_t gid = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t j = gid / kLanesPerLm;
    const int k = (int)(gid % kLanesPerLm);
    const bool lm_ok = j < (uint32_t)A.K;          // whole groups share j: shuffles stay in the group
    const uint64_t o = (uint64_t)j * A.M + k;
    const int cam = (lm_ok && k < A.M) ? A.obs_cam[o] : -1;
    const double f = A.focal[0];
    double p[3] = {0.0, 0.0, 1.0};
    if (lm_ok)
        for (int u = 0; u < 3; ++u) p[u] = A.landmarks[3 * (uint64_t)j + u];
    double uv[2] = {0.0, 0.0};
    if (cam >= 0) uv[0] = A.obs_uv[2 * o], uv[1] = A.obs_uv[2 * o + 1];
    double *Q = A.lm_rec + (uint64_t)(lm_ok ? j : 0) * kBaLmStride;
    if (flags & kUpdate) {
        // p -= H^-1 (g_p + b_f df + sum_o Jp^T (Jx dc)), at the poses and focal length before the step
        const int slot = cam >= 0 ? A.free_slot[cam] : -1;
        double q[12];
#pragma unroll
        for (int t = 0; t < 12; ++t) q[t] = Q[kQH + t];   // H^-1, b_f, g_p
        double v[3] = {0.0, 0.0, 0.0};
        if (slot >= 0) {
            const double *T = A.pose_old + 12 * slot, *dc = A.dc + 6 * slot;
            const ObsGeom g = observe(T, p, A.pose_old[12 * (uint64_t)A.F]);
            double x0[6], x1[6], p0[3], p1[3], e0 = 0.0, e1 = 0.0;
            pose_rows(g, x0, x1);
            point_rows(g, T, p0, p1);
#pragma unroll
            for (int i = 0; i < 6; ++i) e0 = fma(x0[i], dc[i], e0), e1 = fma(x1[i], dc[i], e1);
#pragma unroll
            for (int u = 0; u < 3; ++u) v[u] = fma(p0[u], e0, p1[u] * e1);
        }
        const double df = A.dc[A.D - 1];
        double d[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) v[u] = q[9 + u] + fma(q[6 + u], df, group_sum(v[u]));
        sym3(q, v, d);
#pragma unroll
        for (int u = 0; u < 3; ++u) p[u] -= d[u];
        if (lm_ok && k == 0)
            for (int u = 0; u < 3; ++u) A.landmarks[3 * (uint64_t)j + u] = p[u];
    }
    double r0 = 0.0, r1 = 0.0, xn = 0.0, yn = 0.0, p0[3] = {0.0, 0.0, 0.0}, p1[3] = {0.0, 0.0, 0.0};
    if (cam >= 0) {
        const double *T = A.poses + 12 * (uint64_t)cam;
        const ObsGeom g = observe(T, p, f);
        point_rows(g, T, p0, p1);
        xn = g.xn, yn = g.yn;
        r0 = fma(f, xn, A.cx) - uv[0];
        r1 = fma(f, yn, A.cy) - uv[1];
    }
    // per landmark, on lane 0 of its group: Jf^T Jf, y_f . b_f, Jf^T r - y_f . g_p and the cost,
    // summed over the block's landmarks
    double sums[4];
    const double cost = group_sum(0.5 * (r0 * r0 + r1 * r1));
    const bool first = lm_ok && k == 0;
    sums[3] = first ? cost : 0.0;
    if (flags & kCostOnly) {
        sums[0] = sums[1] = sums[2] = 0.0;
    } else {
        // landmark block, gradient and focal coupling, summed over the group
        double H[6], gp[3], bf[3];
        int t = 0;
#pragma unroll
        for (int u = 0; u < 3; ++u)
#pragma unroll
            for (int v = u; v < 3; ++v) H[t++] = group_sum(fma(p0[u], p0[v], p1[u] * p1[v]));
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            gp[u] = group_sum(fma(p0[u], r0, p1[u] * r1));
            bf[u] = group_sum(fma(xn, p0[u], yn * p1[u]));
        }
        const double ff = group_sum(fma(xn, xn, yn * yn));
        const double sfj = group_sum(fma(xn, r0, yn * r1));
        // H = [[H0 H1 H2], [H1 H3 H4], [H2 H4 H5]], damped; inverse by cofactors
        const double d0 = H[0] * (1.0 + A.lambda), d1 = H[3] * (1.0 + A.lambda), d2 = H[5] * (1.0 + A.lambda);
        const double c00 = d1 * d2 - H[4] * H[4], c01 = H[2] * H[4] - H[1] * d2, c02 = H[1] * H[4] - H[2] * d1;
        const double c11 = d0 * d2 - H[2] * H[2], c12 = H[1] * H[2] - d0 * H[4], c22 = d0 * d1 - H[1] * H[1];
        const double det = d0 * c00 + H[1] * c01 + H[2] * c02;
        const double id = det != 0.0 ? 1.0 / det : 0.0;
        const double hi[6] = {c00 * id, c01 * id, c02 * id, c11 * id, c12 * id, c22 * id};
        double yf[3];
        sym3(hi, bf, yf);
        if (first) {
#pragma unroll
            for (int u = 0; u < 3; ++u) Q[kQP + u] = p[u], Q[kQB + u] = bf[u], Q[kQG + u] = gp[u];
#pragma unroll
            for (int u = 0; u < 6; ++u) Q[kQH + u] = hi[u];
        }
        sums[0] = first ? ff : 0.0;
        sums[1] = first ? dot3(yf, bf) : 0.0;
        sums[2] = first ? sfj - dot3(yf, gp) : 0.0;
    }
    const double *sum = block_sum<kBaThreads / 64>(sums, red);
    if (threadIdx.x < 4) A.lm_sum[4 * (uint64_t)blockIdx.x + threadIdx.x] = sum[threadIdx.x];
}

// Blocks x = 0 .. nblk-1: block (a, b) of the reduced system from its list;
// block x = nblk: the focal-length diagonal entry, its right-hand side and the
// cost.  Each is split over kBaAsmSplit workgroups (y) that take consecutive
// parts of the list (of the landmark blocks) and write a partial system of
// their own; the solve adds the partials in order.
__global__ void __launch_bounds__(kAsmThreads) k_ba_assemble(BaArgs A) {
    __shared__ double red[(kAsmThreads / 64 + 1) * 40];
    const int D = A.D, SP = D + 1, fcol = D - 1;
    const int part = blockIdx.y;
    double *S = A.S + part * part_stride(D), *s = S + (uint64_t)D * SP;
    if ((int)blockIdx.x == A.nblk) {
        const int nb = (A.K + kLmPerBlock - 1) / kLmPerBlock;
        const int i0 = (int)((int64_t)nb * part / kBaAsmSplit), i1 = (int)((int64_t)nb * (part + 1) / kBaAsmSplit);
        double acc[4] = {0.0, 0.0, 0.0, 0.0};
        for (int i = i0 + threadIdx.x; i < i1; i += kAsmThreads)
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] += A.lm_sum[4 * (uint64_t)i + t];
        const double *sum = block_sum<kAsmThreads / 64>(acc, red);
        if (threadIdx.x == 0) {
            S[(uint64_t)fcol * SP + fcol] = sum[0] * (1.0 + A.lambda) - sum[1];
            s[fcol] = sum[2];
            s[D] = sum[3];   // the cost slot after the right-hand side
        }
        return;
    }
    const int2 ab = A.block_ab[blockIdx.x];
    const uint32_t b0 = A.block_off[blockIdx.x], len = A.block_off[blockIdx.x + 1] - b0;
    const uint32_t e0 = b0 + (uint32_t)((uint64_t)len * part / kBaAsmSplit);
    const uint32_t e1 = b0 + (uint32_t)((uint64_t)len * (part + 1) / kBaAsmSplit);
    const int ra = 6 * ab.x, rb = 6 * ab.y;
    const double f = A.focal[0];
    const double *Ta = A.poses + 12 * (uint64_t)A.slot_cam[ab.x];
    if (ab.x == ab.y) {
        // 21 entries of the upper triangle, 6 of diag(Jx^T Jx), the focal column and the right-hand side
        double acc[39];
#pragma unroll
        for (int t = 0; t < 39; ++t) acc[t] = 0.0;
        for (uint32_t e = e0 + threadIdx.x; e < e1; e += kAsmThreads) {
            const uint32_t o = A.pairs[e];
            const double *Q = A.lm_rec + (uint64_t)(o / (uint32_t)A.M) * kBaLmStride;
            double q[15];
#pragma unroll
            for (int t = 0; t < 15; ++t) q[t] = Q[t];
            const double u0 = A.obs_uv[2 * (uint64_t)o], u1 = A.obs_uv[2 * (uint64_t)o + 1];
            const ObsGeom g = observe(Ta, q + kQP, f);
            double x0[6], x1[6], p0[3], p1[3], h0[3], h1[3];
            pose_rows(g, x0, x1);
            point_rows(g, Ta, p0, p1);
            sym3(q + kQH, p0, h0);
            sym3(q + kQH, p1, h1);
            const double m00 = 1.0 - dot3(p0, h0), m01 = -dot3(p0, h1), m11 = 1.0 - dot3(p1, h1);
            const double r0 = fma(f, g.xn, A.cx) - u0, r1 = fma(f, g.yn, A.cy) - u1;
            const double c0 = g.xn - dot3(h0, q + kQB), c1 = g.yn - dot3(h1, q + kQB);
            const double s0 = r0 - dot3(h0, q + kQG), s1 = r1 - dot3(h1, q + kQG);
            int t = 0;
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const double y0 = fma(m00, x0[i], m01 * x1[i]), y1 = fma(m01, x0[i], m11 * x1[i]);
#pragma unroll
                for (int w = i; w < 6; ++w, ++t) acc[t] = fma(y0, x0[w], fma(y1, x1[w], acc[t]));
            }
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                acc[21 + i] = fma(x0[i], x0[i], fma(x1[i], x1[i], acc[21 + i]));
                acc[27 + i] = fma(x0[i], c0, fma(x1[i], c1, acc[27 + i]));
                acc[33 + i] = fma(x0[i], s0, fma(x1[i], s1, acc[33 + i]));
            }
        }
        const double *sum = block_sum<kAsmThreads / 64>(acc, red);
        for (int t = threadIdx.x; t < 36; t += kAsmThreads) {
            const int i = t / 6, q = t % 6;
            const int lo = i < q ? i : q, hi = i < q ? q : i;
            const int tri = lo * 6 - lo * (lo - 1) / 2 + (hi - lo);   // packed upper-triangle index
            double v = sum[tri];
            if (i == q) v += A.lambda * sum[21 + i];
            S[(uint64_t)(ra + i) * SP + ra + q] = v;
        }
        if (threadIdx.x < 6) {
            const int i = threadIdx.x;
            S[(uint64_t)fcol * SP + ra + i] = sum[27 + i];
            s[ra + i] = sum[33 + i];
        }
        return;
    }
    double acc[36];
#pragma unroll
    for (int t = 0; t < 36; ++t) acc[t] = 0.0;
    const double *Tb = A.poses + 12 * (uint64_t)A.slot_cam[ab.y];
    for (uint32_t e = e0 + threadIdx.x; e < e1; e += kAsmThreads) {
        const double *Q = A.lm_rec + (uint64_t)A.pairs[e] * kBaLmStride;
        double q[9];
#pragma unroll
        for (int t = 0; t < 9; ++t) q[t] = Q[t];
        const ObsGeom ga = observe(Ta, q + kQP, f), gb = observe(Tb, q + kQP, f);
        double a0[3], a1[3], p0[3], p1[3], h0[3], h1[3];
        point_rows(ga, Ta, a0, a1);
        point_rows(gb, Tb, p0, p1);
        sym3(q + kQH, p0, h0);
        sym3(q + kQH, p1, h1);
        const double m00 = dot3(a0, h0), m01 = dot3(a0, h1), m10 = dot3(a1, h0), m11 = dot3(a1, h1);
        double x0[6], x1[6], z0[6], z1[6];
        pose_rows(ga, x0, x1);
        pose_rows(gb, z0, z1);
#pragma unroll
        for (int i = 0; i < 6; ++i) {
            const double y0 = fma(m00, x0[i], m10 * x1[i]), y1 = fma(m01, x0[i], m11 * x1[i]);
#pragma unroll
            for (int w = 0; w < 6; ++w) acc[6 * i + w] = fma(y0, z0[w], fma(y1, z1[w], acc[6 * i + w]));
        }
    }
    const double *sum = block_sum<kAsmThreads / 64>(acc, red);
    // (only the lower triangle is read: rows of b, columns of a < b)
    for (int t = threadIdx.x; t < 36; t += kAsmThreads) {
        const int i = t / 6, q = t % 6;
        S[(uint64_t)(rb + q) * SP + ra + i] = -sum[t];
    }
}

// SE(3) exponential of (rho, phi): R = I + a [phi]x + b [phi]x^2,
// V = I + b [phi]x + c [phi]x^2 with a = sin t / t, b = (1 - cos t) / t^2,
// c = (t - sin t) / t^3, t = |phi|.  Up to t = 1/2, where the closed forms of
// b and c cancel, by their power series in t^2 (nine terms: the next is below
// 1e-21), which also keeps the sine and cosine out of the solve's chain.
__device__ void se3_exp(const double xi[6], double Rm[3][3], double tv[3]) {
    const double w0 = xi[3], w1 = xi[4], w2 = xi[5];
    const double t2 = w0 * w0 + w1 * w1 + w2 * w2;
    double a, b, c;
    if (t2 < 0.25) {
        // the k-th coefficients are (-1)^k / (2k + 1)!, / (2k + 2)! and / (2k + 3)!:
        // each ratio to the one before is -1 / ((m - 1) m) for factorial m!
        a = b = c = 1.0;
#pragma unroll
        for (int k = 8; k >= 1; --k) {
            a = fma(-t2 * (1.0 / ((2 * k) * (2 * k + 1))), a, 1.0);
            b = fma(-t2 * (1.0 / ((2 * k + 1) * (2 * k + 2))), b, 1.0);
            c = fma(-t2 * (1.0 / ((2 * k + 2) * (2 * k + 3))), c, 1.0);
        }
        b *= 0.5;
        c *= 1.0 / 6.0;
    } else {
        const double t = sqrt(t2), sn = sin(t), cs = cos(t);
        a = sn / t;
        b = (1.0 - cs) / t2;
        c = (t - sn) / (t2 * t);
    }
    const double W[3][3] = {{0.0, -w2, w1}, {w2, 0.0, -w0}, {-w1, w0, 0.0}};
    double W2[3][3];
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q) W2[r][q] = W[r][0] * W[0][q] + W[r][1] * W[1][q] + W[r][2] * W[2][q];
    double V[3][3];
    for (int r = 0; r < 3; ++r)
        for (int q = 0; q < 3; ++q) {
            const double id = r == q ? 1.0 : 0.0;
            Rm[r][q] = id + a * W[r][q] + b * W2[r][q];
            V[r][q] = id + b * W[r][q] + c * W2[r][q];
        }
    for (int r = 0; r < 3; ++r) tv[r] = V[r][0] * xi[0] + V[r][1] * xi[1] + V[r][2] * xi[2];
}

// v of lane C of this lane's row of 16 (a DPP move: a few cycles, against tens
// for a readlane into a scalar register and back).
template <int C>
__device__ __forceinline__ double row_lane(double v) {
    return __longlong_as_double(
        __builtin_amdgcn_update_dpp((long long)0, (long long)__double_as_longlong(v), 0x150 + C, 0xf, 0xf, true));
}

// f(integral constant I) for I = I0 .. N - 1, for code whose index must be a constant
template <int I>
struct Index {
    static constexpr int value = I;
};
template <int I0, int N, class F>
__device__ __forceinline__ void static_for(F f) {
    if constexpr (I0 < N) {
        f(Index<I0>{});
        static_for<I0 + 1, N>(f);
    }
}

// 1 / d to within about an ulp: the hardware's estimate and two Newton steps.
__device__ __forceinline__ double recip(double d) {
    double y = __builtin_amdgcn_rcp(d);
    y = fma(y, fma(-d, y, 1.0), y);
    return fma(y, fma(-d, y, 1.0), y);
}

// S = L D L^T of the reduced system (D x D, symmetric positive definite after
// damping) in LDS, right-looking in column blocks of 16, with the right-hand
// side s as one more row (row D of the factor is then w^T, w = D^-1 L^-1 s,
// without a forward solve), then L^T dc = -w.  What it costs is the
// serial chain of D pivots, so everything else is taken off it:
//
//   factor + panel  every row of 16 lanes holds the diagonal tile, a row of it
//                   per lane, and each lane one further panel row of the
//                   block's columns, in registers (64 panel rows; the next 64
//                   are another wave's, which factors the diagonal tile again
//                   rather than wait for it).  Column j: the pivot and the
//                   column's entries come from the tile by DPP broadcasts
//                   within the row of lanes, and one reciprocal and one
//                   multiply-add per entry follow; no square root, no LDS and
//                   no scalar register in the chain, and the reciprocal of
//                   the next pivot runs between the updates of this column.
//                   What is left in place is -L.
//   trailing        16 x 16 tiles, C -= L_i D L_j^T, four v_mfma_f64_16x16x4
//                   each, a wave per tile: the next block's column of tiles
//                   at once, the others while waves 0 and 1 factor it.
//
// Two barriers per block of 16 columns.  D = 97: 22.5 us (load 2.3, factor
// and panel 10, trailing 3.3, backward solve 5.1, retraction 0.8) against
// 59 us for a blocked Cholesky by 8 columns with 2 x 2 register tiles.  A
// factoring wave is alone on its SIMD and bound by issue, about 6 cycles an
// FP64 instruction, not by the pivots' dependence (a shorter reciprocal chain
// changed nothing).
__global__ void __launch_bounds__(kSolveThreads) k_ba_solve(BaArgs A, int iter) {
    extern __shared__ __attribute__((aligned(16))) double lds[];
    typedef double v4d __attribute__((ext_vector_type(4)));
    // row pitch 16 NB + 2: 16 rows of one column lie in 16 different bank groups
    const int D = A.D, NB = (D + 1 + kTile - 1) / kTile, N = NB * kTile, P = N + 2;
    double *M = lds, *nd = lds + (size_t)N * P, *dcs = nd + N;   // nd: -D
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int li = lane & 15, lk = lane >> 4;
    const size_t ps = part_stride(D);
    // the lower triangle of the sum of the partial systems (row D: the
    // right-hand side, and the cost in column D), zero in the padding: row
    // wave + 8 i, one 16-byte column pair per lane, every load in flight
    {
        constexpr int W = kSolveThreads / 64, U = kMaxTiles * kTile / W;
        double2 v[U][kBaAsmSplit];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = wave + W * u;
            const bool ok = r <= D && 2 * lane <= r && 2 * lane < D;
#pragma unroll
            for (int q = 0; q < kBaAsmSplit; ++q)
                v[u][q] = ok ? *reinterpret_cast<const double2 *>(A.S + q * ps + (size_t)r * (D + 1) + 2 * lane)
                             : make_double2(0.0, 0.0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int r = wave + W * u;
            if (r >= N || 2 * lane >= N) continue;
            double2 w = v[u][0];
#pragma unroll
            for (int q = 1; q < kBaAsmSplit; ++q) {
                w.x += v[u][q].x;
                w.y += v[u][q].y;
            }
            if (r == D && 2 * lane + 1 == D && A.costs) A.costs[iter] = w.y;
            *reinterpret_cast<double2 *>(M + (size_t)r * P + 2 * lane) = w;
        }
    }
    __syncthreads();
    // tile (ti, tj) of what is left after block kb (ti, tj >= 1 past it)
    const auto trail = [&](int kb, int ti, int tj) {
        const int k0 = kb * kTile, i0 = k0 + kTile * ti, j0 = k0 + kTile * tj;
        const double *Li = M + (size_t)(i0 + li) * P + k0 + lk, *Lj = M + (size_t)(j0 + li) * P + k0 + lk;
        double *C = M + (size_t)(i0 + lk) * P + j0 + li;   // rows 4 apart per register
        v4d acc, ac2 = {0.0, 0.0, 0.0, 0.0};
        double x[4], y[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) x[q] = Li[4 * q] * nd[k0 + 4 * q + lk], y[q] = Lj[4 * q], acc[q] = C[(size_t)(4 * q) * P];
#pragma unroll
        for (int q = 0; q < 2; ++q) {   // two chains of two
            acc = __builtin_amdgcn_mfma_f64_16x16x4f64(x[q], y[q], acc, 0, 0, 0);
            ac2 = __builtin_amdgcn_mfma_f64_16x16x4f64(x[2 + q], y[2 + q], ac2, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) C[(size_t)(4 * q) * P] = acc[q] + ac2[q];
    };
    for (int kb = 0; kb < NB; ++kb) {
        const int k0 = kb * kTile, k1 = k0 + kTile;
        const int rows = D + 1 - k1;   // panel rows below the block (the right-hand side's included)
        const bool mine = wave * 64 < (rows > 1 ? rows : 1);   // (at most waves 0 and 1: D <= 121)
        if (wave >= 2 && kb > 0) {
            // the tiles the previous block left for now
            const int T = NB - kb, left = T * (T - 1) / 2;
            for (int t = wave - 2; t < left; t += kSolveThreads / 64 - 2) {
                int ti = 0, tj = t;
                while (tj > ti) tj -= ++ti;
                trail(kb - 1, ti + 2, tj + 2);
            }
        }
        double a[kTile];
        if (mine) {
            const int r = k1 + wave * 64 + lane;
            const bool in = r <= D;
            const double *top = M + (size_t)(k0 + li) * P + k0, *row = M + (size_t)(in ? r : k0) * P + k0;
            double x[kTile], md = 0.0;
#pragma unroll
            for (int c = 0; c < kTile; c += 2) {
                const double2 w = *reinterpret_cast<const double2 *>(top + c), v = *reinterpret_cast<const double2 *>(row + c);
                a[c] = w.x, a[c + 1] = w.y;
                x[c] = v.x, x[c + 1] = v.y;
            }
            // (columns from D on only change entries nothing reads)
            double inv = recip(row_lane<0>(a[0]));
            static_for<0, kTile>([&](auto J) {
                constexpr int j = decltype(J)::value;
                const double na = -(a[j] * inv), nx = -(x[j] * inv);
                if (li == j) md = -a[j];
                // the next pivot first, then its reciprocal's chain with the
                // other columns' updates between its steps (the compiler keeps
                // the order it is given across the barriers)
                double y = 0.0, e = 0.0, d = 1.0;
                if constexpr (j + 1 < kTile) {
                    const double s = row_lane<j + 1>(a[j]);
                    a[j + 1] = fma(s, na, a[j + 1]);
                    d = row_lane<j + 1>(a[j + 1]);
                    y = __builtin_amdgcn_rcp(d);
                    x[j + 1] = fma(s, nx, x[j + 1]);
                }
                static_for<0, 7>([&](auto U) {
                    constexpr int u = decltype(U)::value, c = j + 2 + 2 * u;
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (c < kTile) {
                        const double s = row_lane<c>(a[j]);
                        a[c] = fma(s, na, a[c]);
                        x[c] = fma(s, nx, x[c]);
                    }
                    if constexpr (c + 1 < kTile) {
                        const double s = row_lane<c + 1>(a[j]);
                        a[c + 1] = fma(s, na, a[c + 1]);
                        x[c + 1] = fma(s, nx, x[c + 1]);
                    }
                    if constexpr (j + 1 < kTile && (u == 0 || u == 2)) e = fma(-d, y, 1.0);
                    if constexpr (j + 1 < kTile && (u == 1 || u == 3)) y = fma(y, e, y);
                    __builtin_amdgcn_sched_barrier(0);
                });
                a[j] = na, x[j] = nx;
                inv = y;
            });
            // (computed here by every lane: sunk into the branch below, the
            // panel's updates would keep all the broadcasts alive)
#pragma unroll
            for (int c = 0; c < kTile; ++c) asm volatile("" : "+v"(x[c]));
            if (in) {
#pragma unroll
                for (int c = 0; c < kTile; c += 2)
                    *reinterpret_cast<double2 *>(M + (size_t)r * P + k0 + c) = make_double2(x[c], x[c + 1]);
            }
            if (wave == 0 && lane < kTile) nd[k0 + lane] = md;
        }
        __syncthreads();
        // the diagonal tile, which every panel wave has read by now
        if (wave == 0 && lane < kTile) {
#pragma unroll
            for (int c = 0; c < kTile; c += 2)
                *reinterpret_cast<double2 *>(M + (size_t)(k0 + lane) * P + k0 + c) = make_double2(a[c], a[c + 1]);
        }
        if (wave < NB - 1 - kb) trail(kb, wave + 1, 1);   // the next block's column of tiles
        __syncthreads();
    }
    // L^T dc = -w by wave 0, from the last block up; lane owns entries lane
    // and lane + 64.  A block's 16 entries are solved in every row of 16 lanes
    // alike (its rows of -L, a column per lane, and DPP broadcasts), then
    // folded into the entries above it.
    if (wave != 0) return;
    double T[12];   // the pose lane a < F retracts: its load overlaps the solve
    if (lane < A.F)
        for (int q = 0; q < 12; ++q) T[q] = A.poses[12 * (uint64_t)A.slot_cam[lane] + q];
    const int c0 = lane, c1 = lane + 64, a0 = c0 < N ? c0 : N - 1, a1 = c1 < N ? c1 : N - 1;
    double y0 = M[(size_t)D * P + a0], y1 = M[(size_t)D * P + a1];
    if (c0 < D) dcs[c0] = y0;
    if (c1 < D) dcs[c1] = y1;
    double lt[kTile];
#pragma unroll
    for (int u = 0; u < kTile; ++u) lt[u] = M[(size_t)((NB - 1) * kTile + u) * P + (NB - 1) * kTile + li];
    for (int kb = NB - 1; kb >= 0; --kb) {
        const int k0 = kb * kTile;
        const bool valid = k0 + li < D, two = k0 > 64;   // (entries 64.. only matter to blocks beyond them)
        double m0[kTile], m1[kTile];
        double x = valid ? dcs[k0 + li] : 0.0;
#pragma unroll
        for (int u = 0; u < kTile; ++u) m0[u] = M[(size_t)(k0 + u) * P + a0];
        if (two)
#pragma unroll
            for (int u = 0; u < kTile; ++u) m1[u] = M[(size_t)(k0 + u) * P + a1];
#pragma unroll
        for (int u = 1; u < kTile; ++u) lt[u] = (valid & (li < u)) ? lt[u] : 0.0;   // (entries beyond may be anything)
        static_for<0, kTile - 1>([&](auto U) {
            constexpr int u = kTile - 1 - decltype(U)::value;
            x = fma(lt[u], row_lane<u>(x), x);
        });
        if (lane < kTile && valid) dcs[k0 + lane] = x;
        if (kb > 0)   // the next block's, ahead of its use
#pragma unroll
            for (int u = 0; u < kTile; ++u) lt[u] = M[(size_t)(k0 - kTile + u) * P + k0 - kTile + li];
        double s0 = 0.0;
        static_for<0, kTile / 2>([&](auto U) {
            constexpr int u = 2 * decltype(U)::value;
            y0 = fma(m0[u], row_lane<u>(x), y0);
            s0 = fma(m0[u + 1], row_lane<u + 1>(x), s0);
        });
        y0 += s0;   // (of use to the entries above the block only)
        if (c0 < k0) dcs[c0] = y0;
        if (two) {
            double s1 = 0.0;
            static_for<0, kTile / 2>([&](auto U) {
                constexpr int u = 2 * decltype(U)::value;
                y1 = fma(m1[u], row_lane<u>(x), y1);
                s1 = fma(m1[u + 1], row_lane<u + 1>(x), s1);
            });
            y1 += s1;
            if (c1 < k0) dcs[c1] = y1;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    if (c0 < D) A.dc[c0] = dcs[c0];
    if (c1 < D) A.dc[c1] = dcs[c1];
    // T_a <- exp(dc_a) T_a and f += df; the poses and the focal length before
    // the step stay in pose_old for the landmark update
    if (lane < A.F) {
        double xi[6], Rm[3][3], tv[3];
        for (int q = 0; q < 6; ++q) xi[q] = dcs[6 * lane + q];
        se3_exp(xi, Rm, tv);
        double *now = A.poses + 12 * (uint64_t)A.slot_cam[lane], *old = A.pose_old + 12 * lane;
        for (int q = 0; q < 12; ++q) old[q] = T[q];
        for (int r = 0; r < 3; ++r)
            for (int q = 0; q < 4; ++q)
                now[4 * r + q] = Rm[r][0] * T[q] + Rm[r][1] * T[4 + q] + Rm[r][2] * T[8 + q] + (q == 3 ? tv[r] : 0.0);
    }
    if (lane == 63) {
        const double f = A.focal[0];
        A.pose_old[12 * (uint64_t)A.F] = f;
        A.focal[0] = f + dcs[D - 1];
    }
}

__global__ void __launch_bounds__(kBaThreads) k_ba_cost(BaArgs A, int iter) {
    __shared__ double red[5 * 4];
    const int nb = (A.K + kLmPerBlock - 1) / kLmPerBlock;
    double acc[1] = {0.0};
    for (int i0 = threadIdx.x; i0 < nb; i0 += 4 * kBaThreads) {   // 4 loads in flight per thread
        double v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int i = i0 + u * kBaThreads;
            v[u] = i < nb ? A.lm_sum[4 * (uint64_t)i + 3] : 0.0;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) acc[0] += v[u];
    }
    const double *sum = block_sum<kBaThreads / 64>(acc, red);
    if (threadIdx.x == 0 && A.costs) A.costs[iter] = sum[0];
}

}  // namespace

size_t ba_lds_bytes(int D) {
    const size_t N = (size_t)(D + 1 + kTile - 1) / kTile * kTile;
    return (N * (N + 2) + 2 * N) * sizeof(double);
}

hipError_t ba_allow_lds(int D) {
    return hipFuncSetAttribute(reinterpret_cast<const void *>(&k_ba_solve), hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)ba_lds_bytes(D));
}

size_t ba_lm_blocks(int K) { return ((size_t)K + kLmPerBlock - 1) / kLmPerBlock; }

void launch_ba_iterations(const BaArgs &A, int iterations, hipStream_t st) {
    const unsigned lm_blocks = (unsigned)ba_lm_blocks(A.K);
    const size_t solve_lds = ba_lds_bytes(A.D);
    for (int it = 0; it < iterations; ++it) {
        hipLaunchKernelGGL(k_ba_landmark, dim3(lm_blocks), dim3(kBaThreads), 0, st, A, it > 0 ? kUpdate : 0);
        hipLaunchKernelGGL(k_ba_assemble, dim3((unsigned)A.nblk + 1, kBaAsmSplit), dim3(kAsmThreads), 0, st, A);
        hipLaunchKernelGGL(k_ba_solve, dim3(1), dim3(kSolveThreads), solve_lds, st, A, it);
    }
    hipLaunchKernelGGL(k_ba_landmark, dim3(lm_blocks), dim3(kBaThreads), 0, st, A, (iterations > 0 ? kUpdate : 0) | kCostOnly);
    hipLaunchKernelGGL(k_ba_cost, dim3(1), dim3(kBaThreads), 0, st, A, iterations);
}

}  // namespace gsr
