// gsr_update.hip -- parameter updates around the rasterizer on gfx950:
//   * the fused Adam step of the joint optimisation over the five Gaussian
//     arrays (optionally only for the Gaussians the last forward saw),
//   * the pose step: Adam on each view's 6-DoF twist, then the SE(3)
//     retraction of its world-to-camera transform,
//   * the loop-closure Sim(3) relocation of Gaussians (or hierarchy nodes).
// The first and last are elementwise and HBM-bound: every array is walked as
// one flat sequence of float4 (or float) units, so loads and stores are
// coalesced whatever the row length of an array (but for the sparse Adam step of
// mid-sized calls, which walks the rows of listed Gaussians).
#include <algorithm>

#include "gsr_internal.h"

namespace gsr {

constexpr float kOpacityLo = 1e-7f, kOpacityHi = 1.f - 1e-7f;

// Did some view of the last forward see Gaussian i?  (count = tiles touched)
__device__ __forceinline__ bool seen(const uint32_t *__restrict__ count, uint64_t n, int n_views, uint64_t i) {
    bool s = false;
    for (int v = 0; v < n_views; ++v) s |= count[(uint64_t)v * n + i] > 0u;
    return s;
}

__device__ __forceinline__ void adam_elem(float &p, float g, float &m, float &v, const AdamScalars &a, float step_size) {
    m = fmaf(a.b1, m, a.one_m_b1 * g);
    v = fmaf(a.b2, v, a.one_m_b2 * g * g);
    const float denom = fmaf(sqrtf(v), a.inv_sqrt_bc2, a.eps);
    p -= step_size * (m / denom);
}

// One array of the parameter set, as flat float (W = 1) or float4 (W = 4) units.
template <int W>
__device__ __forceinline__ void adam_units(float *p, const float *g, float *m, float *v, uint64_t unit,
                                           const AdamScalars &a, float step_size) {
    if constexpr (W == 4) {
        float4 P = reinterpret_cast<float4 *>(p)[unit], G = reinterpret_cast<const float4 *>(g)[unit];
        float4 M = reinterpret_cast<float4 *>(m)[unit], V = reinterpret_cast<float4 *>(v)[unit];
        adam_elem(P.x, G.x, M.x, V.x, a, step_size);
        adam_elem(P.y, G.y, M.y, V.y, a, step_size);
        adam_elem(P.z, G.z, M.z, V.z, a, step_size);
        adam_elem(P.w, G.w, M.w, V.w, a, step_size);
        reinterpret_cast<float4 *>(p)[unit] = P;
        reinterpret_cast<float4 *>(m)[unit] = M;
        reinterpret_cast<float4 *>(v)[unit] = V;
    } else {
        float P = p[unit], M = m[unit], V = v[unit];
        adam_elem(P, g[unit], M, V, a, step_size);
        p[unit] = P;
        m[unit] = M;
        v[unit] = V;
    }
}

// Segments of the flat walk: means (3n floats), log-scales (3n floats),
// quaternions (n float4), opacities (n floats, on the logit), SH (n 3K/4
// float4 when 3K is a multiple of 4, else n 3K floats).
//
// HBM-bound: 28 bytes a parameter (four read, three written), each array one ascending sweep.  The row
// length is a constant and the unit index 32 bits wide wherever it fits: finding
// a unit's Gaussian and its place in the row by 64-bit division by a variable
// bound the smaller calls: 30 k Gaussians of degree 3 7.8 -> 7.2 us, 300 k of
// degree 2 51.4 -> 49.8 us, 1 M as before (307 and 192 -> 188 us).
template <int K, typename U>
__global__ __launch_bounds__(256) void k_adam_step(AdamArgs A) {
    constexpr bool kVec = (3 * K) % 4 == 0;
    constexpr U kUnits = kVec ? 3 * K / 4 : 3 * K;  // units per SH row
    const U n = (U)A.n, s0 = 3 * n, s1 = s0 + 3 * n, s2 = s1 + n, s3 = s2 + n, total = s3 + n * kUnits;
    const U stride = (U)gridDim.x * 256;
    for (U u = (U)blockIdx.x * 256 + threadIdx.x; u < total; u += stride) {
        // Gaussian of this unit
        const U gi = u < s0 ? u / 3 : u < s1 ? (u - s0) / 3 : u < s2 ? u - s1 : u < s3 ? u - s2 : (u - s3) / kUnits;
        if (A.count && !seen(A.count, A.n, A.n_views, gi)) continue;
        if (u < s0) {
            adam_units<1>(A.p.means, A.g.means, A.m.means, A.v.means, u, A.a, A.step_size[0]);
        } else if (u < s1) {
            adam_units<1>(A.p.log_scales, A.g.log_scales, A.m.log_scales, A.v.log_scales, u - s0, A.a,
                          A.step_size[1]);
        } else if (u < s2) {
            adam_units<4>(A.p.quats, A.g.quats, A.m.quats, A.v.quats, u - s1, A.a, A.step_size[2]);
        } else if (u < s3) {
            // opacity: the step is on l = ln(o / (1 - o)), with dL/dl = o (1 - o) dL/do
            const U i = u - s2;
            const float o = fminf(fmaxf(A.p.opacities[i], kOpacityLo), kOpacityHi);
            float l = logf(o) - log1pf(-o);
            float m = A.m.opacities[i], v = A.v.opacities[i];
            adam_elem(l, o * (1.f - o) * A.g.opacities[i], m, v, A.a, A.step_size[3]);
            A.p.opacities[i] = 1.f / (1.f + expf(-l));
            A.m.opacities[i] = m;
            A.v.opacities[i] = v;
        } else {
            const U w = u - s3, c = w - gi * kUnits;  // unit of the row
            if constexpr (kVec) {
                // (the first unit of a row holds the three DC floats and one float of k = 1)
                const float rate = A.step_size[5], first = c == 0 ? A.step_size[4] : rate;
                float4 P = reinterpret_cast<float4 *>(A.p.sh)[w], G = reinterpret_cast<const float4 *>(A.g.sh)[w];
                float4 M = reinterpret_cast<float4 *>(A.m.sh)[w], V = reinterpret_cast<float4 *>(A.v.sh)[w];
                adam_elem(P.x, G.x, M.x, V.x, A.a, first);
                adam_elem(P.y, G.y, M.y, V.y, A.a, first);
                adam_elem(P.z, G.z, M.z, V.z, A.a, first);
                adam_elem(P.w, G.w, M.w, V.w, A.a, rate);
                reinterpret_cast<float4 *>(A.p.sh)[w] = P;
                reinterpret_cast<float4 *>(A.m.sh)[w] = M;
                reinterpret_cast<float4 *>(A.v.sh)[w] = V;
            } else {
                adam_units<1>(A.p.sh, A.g.sh, A.m.sh, A.v.sh, w, A.a, c < 3 ? A.step_size[4] : A.step_size[5]);
            }
        }
    }
}

// The sparse step of mid-sized calls: a workgroup takes 64 Gaussians, lists the
// ones some view saw and walks their rows with every lane busy, the SH rows by
// the whole workgroup, the other arrays by a wave each.
constexpr int kAdamGroup = 64;
constexpr uint64_t kAdamListMin = 32768, kAdamListSpan = 512ull << 20;
template <int K>
__global__ __launch_bounds__(256) void k_adam_listed(AdamArgs A) {
    constexpr bool kVec = (3 * K) % 4 == 0;
    constexpr uint32_t kW = kVec ? 4 : 1, kUnits = 3 * K / kW;  // floats a unit; units an SH row
    __shared__ uint8_t list[kAdamGroup];
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint64_t base = (uint64_t)blockIdx.x * kAdamGroup;
    const bool on = base + lane < A.n && seen(A.count, A.n, A.n_views, base + lane);
    const unsigned long long m = __ballot(on);
    if (wave == 0 && on) list[__popcll(m & ((1ull << lane) - 1ull))] = (uint8_t)lane;
    __syncthreads();
    const uint32_t rows = (uint32_t)__popcll(m);
#pragma unroll 2
    for (uint32_t u = threadIdx.x; u < rows * kUnits; u += 256) {
        const uint32_t r = u / kUnits, c = u - r * kUnits;
        const uint64_t w = (base + list[r]) * kUnits + c;
        if constexpr (kVec) {
            // (the first unit of a row holds the three DC floats and one float of k = 1)
            const float rate = A.step_size[5], first = c == 0 ? A.step_size[4] : rate;
            float4 P = reinterpret_cast<float4 *>(A.p.sh)[w], G = reinterpret_cast<const float4 *>(A.g.sh)[w];
            float4 M = reinterpret_cast<float4 *>(A.m.sh)[w], V = reinterpret_cast<float4 *>(A.v.sh)[w];
            adam_elem(P.x, G.x, M.x, V.x, A.a, first);
            adam_elem(P.y, G.y, M.y, V.y, A.a, first);
            adam_elem(P.z, G.z, M.z, V.z, A.a, first);
            adam_elem(P.w, G.w, M.w, V.w, A.a, rate);
            reinterpret_cast<float4 *>(A.p.sh)[w] = P;
            reinterpret_cast<float4 *>(A.m.sh)[w] = M;
            reinterpret_cast<float4 *>(A.v.sh)[w] = V;
        } else {
            adam_units<1>(A.p.sh, A.g.sh, A.m.sh, A.v.sh, w, A.a, c < 3 ? A.step_size[4] : A.step_size[5]);
        }
    }
    if (wave < 2) {  // means, log-scales
        for (uint32_t u = lane; u < 3 * rows; u += kWave) {
            const uint32_t r = u / 3;
            const uint64_t e = (base + list[r]) * 3 + (u - 3 * r);
            if (wave == 0)
                adam_units<1>(A.p.means, A.g.means, A.m.means, A.v.means, e, A.a, A.step_size[0]);
            else
                adam_units<1>(A.p.log_scales, A.g.log_scales, A.m.log_scales, A.v.log_scales, e, A.a, A.step_size[1]);
        }
    } else if (lane < rows) {
        const uint64_t i = base + list[lane];
        if (wave == 2) {
            adam_units<4>(A.p.quats, A.g.quats, A.m.quats, A.v.quats, i, A.a, A.step_size[2]);
        } else {
            // opacity: the step is on l = ln(o / (1 - o)), with dL/dl = o (1 - o) dL/do
            const float o = fminf(fmaxf(A.p.opacities[i], kOpacityLo), kOpacityHi);
            float l = logf(o) - log1pf(-o);
            float mo = A.m.opacities[i], vo = A.v.opacities[i];
            adam_elem(l, o * (1.f - o) * A.g.opacities[i], mo, vo, A.a, A.step_size[3]);
            A.p.opacities[i] = 1.f / (1.f + expf(-l));
            A.m.opacities[i] = mo;
            A.v.opacities[i] = vo;
        }
    }
}

template <int K>
static void launch_adam(const AdamArgs &A, hipStream_t st) {
    // The lanes of unseen Gaussians cost the flat walk most of its time, but from
    // about half a gigabyte of arrays on (parameters, gradients, moments) five
    // ascending sweeps use the memory better than runs of rows dealt over all of
    // them.  Listed and flat: 400 k (378 MB, 191 k seen) 73 / 78 us, 560 k (529 MB)
    // 80.5 / 99 us, 700 k (661 MB) 125.3 / 124.3 us, 1 M (944 MB, 478 k seen) 251 /
    // 235 us; 20 k Gaussians 6.1 / 5.1 us.  With every Gaussian seen, which the host
    // cannot know, 400 k take 124 / 121 us (degree 2: 64 / 74), with few 12 / 23 us.
    const uint64_t span = A.n * (11 + 3 * K) * 16;
    if (A.count && A.n >= kAdamListMin && span <= kAdamListSpan) {
        hipLaunchKernelGGL(k_adam_listed<K>, dim3((unsigned)((A.n + kAdamGroup - 1) / kAdamGroup)), dim3(256), 0, st, A);
        return;
    }
    constexpr uint64_t kUnits = (3 * K) % 4 == 0 ? 3 * K / 4 : 3 * K;
    const uint64_t total = A.n * (8 + kUnits), blocks = std::min<uint64_t>((total + 255) / 256, 65536);
    // (an index that steps past the end by a stride must not wrap)
    if (total + blocks * 256 < (1ull << 32))
        hipLaunchKernelGGL((k_adam_step<K, uint32_t>), dim3((unsigned)blocks), dim3(256), 0, st, A);
    else
        hipLaunchKernelGGL((k_adam_step<K, uint64_t>), dim3((unsigned)blocks), dim3(256), 0, st, A);
}

void launch_adam_step(const AdamArgs &A, hipStream_t st) {
    if (A.n == 0) return;
    switch (A.sh_k) {
        case 1: launch_adam<1>(A, st); break;
        case 4: launch_adam<4>(A, st); break;
        case 9: launch_adam<9>(A, st); break;
        default: launch_adam<16>(A, st); break;
    }
}

// ---------------------------------------------------------------------------
// Pose step: one thread per view.  xi = -lr m_hat / (sqrt(v_hat) + eps), then
// T <- exp(xi^) T with the closed-form SE(3) exponential: for phi = xi[3:6],
// theta = |phi|, R = I + a [phi]x + b [phi]x^2 and t = (I + b [phi]x + c [phi]x^2) rho
// with a = sin(theta)/theta, b = (1 - cos(theta))/theta^2,
// c = (theta - sin(theta))/theta^3 (series near theta = 0).
// ---------------------------------------------------------------------------
__global__ void k_pose_step(float *__restrict__ w2c, const float *__restrict__ g, float *__restrict__ m,
                            float *__restrict__ v, int n_views, AdamScalars a, float step_size) {
    const int k = threadIdx.x;
    if (k >= n_views) return;
    double xi[6];
#pragma unroll
    for (int j = 0; j < 6; ++j) {
        float p = 0.f, mj = m[6 * k + j], vj = v[6 * k + j];
        adam_elem(p, g[6 * k + j], mj, vj, a, step_size);
        m[6 * k + j] = mj;
        v[6 * k + j] = vj;
        xi[j] = (double)p;
    }
    const double px = xi[3], py = xi[4], pz = xi[5];
    const double th2 = px * px + py * py + pz * pz, th = sqrt(th2);
    double ca, cb, cc;
    if (th < 1e-4) {
        ca = 1.0 - th2 / 6.0;
        cb = 0.5 - th2 / 24.0;
        cc = 1.0 / 6.0 - th2 / 120.0;
    } else {
        ca = sin(th) / th;
        cb = (1.0 - cos(th)) / th2;
        cc = (th - sin(th)) / (th2 * th);
    }
    const double W[9] = {0, -pz, py, pz, 0, -px, -py, px, 0};
    double W2[9];
    for (int r = 0; r < 3; ++r)
        for (int c = 0; c < 3; ++c) W2[3 * r + c] = W[3 * r] * W[c] + W[3 * r + 1] * W[3 + c] + W[3 * r + 2] * W[6 + c];
    double E[16];
    for (int r = 0; r < 3; ++r) {
        double t = 0.0;
        for (int c = 0; c < 3; ++c) {
            const double id = r == c ? 1.0 : 0.0;
            E[4 * r + c] = id + ca * W[3 * r + c] + cb * W2[3 * r + c];
            t += (id + cb * W[3 * r + c] + cc * W2[3 * r + c]) * xi[c];
        }
        E[4 * r + 3] = t;
    }
    E[12] = E[13] = E[14] = 0.0;
    E[15] = 1.0;
    float *T = w2c + 16 * k;
    double Tin[16];
    for (int j = 0; j < 16; ++j) Tin[j] = (double)T[j];
    for (int r = 0; r < 4; ++r)
        for (int c = 0; c < 4; ++c) {
            double s = 0.0;
            for (int j = 0; j < 4; ++j) s += E[4 * r + j] * Tin[4 * j + c];
            T[4 * r + c] = (float)s;
        }
}

void launch_pose_step(float *w2c, const float *g, float *m, float *v, int n_views, const AdamScalars &a,
                      float step_size, hipStream_t st) {
    hipLaunchKernelGGL(k_pose_step, dim3(1), dim3(64), 0, st, w2c, g, m, v, n_views, a, step_size);
}

// ---------------------------------------------------------------------------
// Sim(3) relocation: one thread per Gaussian.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_sim3_relocate(float *__restrict__ means, float *__restrict__ quats,
                                                       float *__restrict__ log_scales, uint64_t n,
                                                       const int32_t *__restrict__ keyframe_of,
                                                       const float *__restrict__ sim3, int32_t n_keyframes) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    const int32_t k = keyframe_of[i];
    if (k < 0 || k >= n_keyframes) return;
    const float *S = sim3 + 8 * (size_t)k;
    const float s = S[0], qw = S[1], qx = S[2], qy = S[3], qz = S[4];
    // R(q) of the unit quaternion (w, x, y, z)
    const float R[9] = {1.f - 2.f * (qy * qy + qz * qz), 2.f * (qx * qy - qw * qz), 2.f * (qx * qz + qw * qy),
                        2.f * (qx * qy + qw * qz), 1.f - 2.f * (qx * qx + qz * qz), 2.f * (qy * qz - qw * qx),
                        2.f * (qx * qz - qw * qy), 2.f * (qy * qz + qw * qx), 1.f - 2.f * (qx * qx + qy * qy)};
    const float mx = means[3 * i], my = means[3 * i + 1], mz = means[3 * i + 2];
    means[3 * i] = fmaf(s, R[0] * mx + R[1] * my + R[2] * mz, S[5]);
    means[3 * i + 1] = fmaf(s, R[3] * mx + R[4] * my + R[5] * mz, S[6]);
    means[3 * i + 2] = fmaf(s, R[6] * mx + R[7] * my + R[8] * mz, S[7]);
    const float4 g = reinterpret_cast<const float4 *>(quats)[i];  // (w, x, y, z)
    reinterpret_cast<float4 *>(quats)[i] =
        make_float4(qw * g.x - qx * g.y - qy * g.z - qz * g.w, qw * g.y + qx * g.x + qy * g.w - qz * g.z,
                    qw * g.z - qx * g.w + qy * g.x + qz * g.y, qw * g.w + qx * g.z - qy * g.y + qz * g.x);
    const float ls = logf(s);
    log_scales[3 * i] += ls;
    log_scales[3 * i + 1] += ls;
    log_scales[3 * i + 2] += ls;
}

void launch_sim3_relocate(float *means, float *quats, float *log_scales, uint64_t n, const int32_t *keyframe_of,
                          const float *sim3, int32_t n_keyframes, hipStream_t st) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_sim3_relocate, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, means, quats,
                       log_scales, n, keyframe_of, sim3, n_keyframes);
}

}  // namespace gsr
