// gsr_hierarchy.hip -- per-view level-of-detail cut of a Gaussian hierarchy
// and the gather of the cut's rows, on gfx950.
//
// Rendering a hierarchy starts from its roots and descends until a node is
// finer than a screen-size threshold or is a leaf (Sec. 7.2); with the screen
// size S = f * (largest axis scale) / (distance to the camera centre), a node
// is in the cut exactly when it does not descend (it is a leaf or S < tau)
// while every one of its ancestors does.  That makes the cut a per-node test:
// one kernel marks the nodes that descend, a second one walks each node's
// ancestor chain (a few levels), and an ordered compaction lists the cut in
// ascending node order.  S is evaluated in double precision so that the
// decision agrees with the FP64 reference away from ties.
#include <algorithm>

#include "gsr_internal.h"

namespace gsr {

constexpr int kMaxDepth = 64;  // longer ancestor chains (or cycles) are cut off

__global__ __launch_bounds__(256) void k_cut_descend(const float *__restrict__ means,
                                                     const float *__restrict__ log_scales,
                                                     const int32_t *__restrict__ child_count, uint64_t n,
                                                     const float *__restrict__ w2c, double focal, double tau,
                                                     uint8_t *__restrict__ descend) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    if (child_count[i] <= 0) {
        descend[i] = 0;
        return;
    }
    // camera centre c = -R^T t of the row-major world-to-camera transform
    double c[3];
    for (int a = 0; a < 3; ++a)
        c[a] = -((double)w2c[a] * w2c[3] + (double)w2c[4 + a] * w2c[7] + (double)w2c[8 + a] * w2c[11]);
    const double dx = (double)means[3 * i] - c[0], dy = (double)means[3 * i + 1] - c[1],
                 dz = (double)means[3 * i + 2] - c[2];
    const double dist = fmax(sqrt(dx * dx + dy * dy + dz * dz), 1e-9);
    const float lmax = fmaxf(fmaxf(log_scales[3 * i], log_scales[3 * i + 1]), log_scales[3 * i + 2]);
    const double s = focal * exp((double)lmax) / dist;
    descend[i] = s >= tau ? 1 : 0;
}

// Four consecutive nodes per thread.  They are mostly siblings, and siblings
// share their ancestors: a chain, a run of dependent gathers whose address
// processing is what bounds the kernel, is walked once for them.  A hop fetches
// the ancestor's flag and its parent together.  4.6 M nodes, 1.4 M of them in
// the cut: 35 us with a thread and a chain per node, 20 us.  Nodes in random order
// have four chains to a thread; workgroups of one wave keep the end of such a launch
// short (whole cuts of 2.3 M and 4.6 M: 119 and 287 us with a node per thread, 137 and
// 302 with four and workgroups of four waves, 132 and 295; in order 39 and 73, 26 and
// 47, 26 and 46; with two nodes random ones take 120 and 284, but ordered ones 28 and 52).
constexpr int kSelectNodes = 4, kSelectThreads = 64;
__global__ __launch_bounds__(kSelectThreads) void k_cut_select(const int32_t *__restrict__ parent, uint64_t n,
                                                               const uint8_t *__restrict__ descend,
                                                               uint8_t *__restrict__ in_cut) {
    const uint64_t i0 = ((uint64_t)blockIdx.x * kSelectThreads + threadIdx.x) * kSelectNodes;
    if (i0 >= n) return;
    const int m = (int)min((uint64_t)kSelectNodes, n - i0);
    uint32_t flags = 0;  // a byte per node (the arrays are scratch: whole words are in bounds and aligned)
    if (m == kSelectNodes)
        flags = *reinterpret_cast<const uint32_t *>(descend + i0);
    else
        for (int q = 0; q < m; ++q) flags |= (uint32_t)descend[i0 + q] << (8 * q);
    int32_t a[kSelectNodes];
#pragma unroll
    for (int q = 0; q < kSelectNodes; ++q) a[q] = q < m ? parent[i0 + q] : -1;
    uint32_t out = 0;
    int64_t walked = INT64_MIN;  // (no 32-bit parent: any negative one marks a root)
    bool all = false;  // every ancestor from `walked` up descends
#pragma unroll
    for (int q = 0; q < kSelectNodes; ++q) {
        if (q >= m || (flags >> (8 * q) & 0xffu)) continue;
        if (a[q] != walked) {
            walked = a[q];
            all = true;
            int64_t at = a[q];
            for (int hop = 0; at >= 0 && (uint64_t)at < n; ++hop) {
                const uint8_t d = descend[at];
                const int32_t up = parent[at];
                if (hop == kMaxDepth || !d) {
                    all = false;
                    break;
                }
                at = up;
            }
        }
        out |= (all ? 1u : 0u) << (8 * q);
    }
    if (m == kSelectNodes)
        *reinterpret_cast<uint32_t *>(in_cut + i0) = out;
    else
        for (int q = 0; q < m; ++q) in_cut[i0 + q] = (uint8_t)(out >> (8 * q));
}

void launch_hierarchy_cut_flags(const float *means, const float *log_scales, const int32_t *parent,
                                const int32_t *child_count, uint64_t n, const float *w2c, float focal, float tau,
                                uint8_t *descend, uint8_t *in_cut, hipStream_t st) {
    if (n == 0) return;
    const dim3 grid((unsigned)((n + 255) / 256));
    hipLaunchKernelGGL(k_cut_descend, grid, dim3(256), 0, st, means, log_scales, child_count, n, w2c, (double)focal,
                       (double)tau, descend);
    constexpr uint64_t per = kSelectThreads * kSelectNodes;
    hipLaunchKernelGGL(k_cut_select, dim3((unsigned)((n + per - 1) / per)), dim3(kSelectThreads), 0, st, parent, n,
                       descend, in_cut);
}

// Row gather as one flat walk over output units (consecutive lanes copy
// consecutive units, so stores are coalesced and, for the ascending runs a cut
// mostly consists of, so are loads): means and log-scales as floats (3 per
// row), quaternions as float4, opacities as floats, SH as float4 when a row is
// a multiple of 16 bytes, else as floats.
template <int K>
__global__ __launch_bounds__(256) void k_gather(gsr_gaussians src, const int32_t *__restrict__ index, uint64_t n_max,
                                                const int64_t *__restrict__ count, gsr_param_set dst) {
    const uint64_t n_out = count ? (uint64_t)min((int64_t)n_max, max(*count, (int64_t)0)) : n_max;
    constexpr bool kVec = (3 * K) % 4 == 0;
    constexpr uint64_t kShUnits = kVec ? 3 * K / 4 : 3 * K;  // SH units per row
    const uint64_t s0 = 3 * n_out, s1 = s0 + 3 * n_out, s2 = s1 + n_out, s3 = s2 + n_out;
    const uint64_t total = s3 + kShUnits * n_out;
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t u = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; u < total; u += stride) {
        if (u < s0) {
            const uint64_t r = u / 3, c = u - 3 * r;
            dst.means[u] = src.means[3 * (uint64_t)index[r] + c];
        } else if (u < s1) {
            const uint64_t w = u - s0, r = w / 3, c = w - 3 * r;
            dst.log_scales[w] = src.log_scales[3 * (uint64_t)index[r] + c];
        } else if (u < s2) {
            const uint64_t r = u - s1;
            reinterpret_cast<float4 *>(dst.quats)[r] = reinterpret_cast<const float4 *>(src.quats)[index[r]];
        } else if (u < s3) {
            const uint64_t r = u - s2;
            dst.opacities[r] = src.opacities[index[r]];
        } else {
            const uint64_t w = u - s3, r = w / kShUnits, c = w - kShUnits * r;
            const uint64_t from = (uint64_t)index[r] * kShUnits + c;
            if constexpr (kVec)
                reinterpret_cast<float4 *>(dst.sh)[w] = reinterpret_cast<const float4 *>(src.sh)[from];
            else
                dst.sh[w] = src.sh[from];
        }
    }
}

void launch_gather_gaussians(const gsr_gaussians &src, const int32_t *index, uint64_t n_out, const int64_t *count,
                             const gsr_param_set &dst, hipStream_t st) {
    if (n_out == 0) return;
    const dim3 grid(4096);  // grid-stride walk
    switch (src.sh_degree) {
        case 0: hipLaunchKernelGGL(k_gather<1>, grid, dim3(256), 0, st, src, index, n_out, count, dst); break;
        case 1: hipLaunchKernelGGL(k_gather<4>, grid, dim3(256), 0, st, src, index, n_out, count, dst); break;
        case 2: hipLaunchKernelGGL(k_gather<9>, grid, dim3(256), 0, st, src, index, n_out, count, dst); break;
        default: hipLaunchKernelGGL(k_gather<16>, grid, dim3(256), 0, st, src, index, n_out, count, dst); break;
    }
}

// The cut's size as the device int64 that gathers and rasterizations read.
__global__ void k_store_count_i64(const uint32_t *__restrict__ count, int64_t *__restrict__ out) {
    if (threadIdx.x == 0) *out = count ? (int64_t)*count : 0;
}

void launch_store_count_i64(const uint32_t *count, int64_t *out, hipStream_t st) {
    hipLaunchKernelGGL(k_store_count_i64, dim3(1), dim3(64), 0, st, count, out);
}


// ---------------------------------------------------------------------------
// Hierarchy build (Sec. 7.1: groups of Gaussians merged into one node by a
// KL-divergence criterion).  Level l + 1 merges runs of `branching`
// consecutive level-l nodes; a parent is the single Gaussian that minimises
// KL(mixture || single) for the opacity-weighted mixture of its children,
// i.e. the mixture's mean and covariance:
//   w_i = o_i / sum o,  mu = sum w_i mu_i,
//   Sigma = sum w_i (Sigma_i + (mu_i - mu)(mu_i - mu)^T),
// with opacity 1 - prod (1 - o_i) and the w-weighted mean of the SH rows.
// The covariance is stored factored: eigenvalues ascending -> log-scales,
// eigenvectors (determinant +1) -> quaternion with w >= 0.
//
// One launch per level (large levels of few children a parent: two); its
// workgroups are of two kinds, dealt in turn so that the arithmetic of one runs
// under the memory traffic of the other.
//
// Geometry, FP64: a thread per child forms its weighted moments (about the
// first child's mean, so the spread term does not cancel against the
// coordinates' magnitude on a street 2 km long), the sums over each parent's
// children are taken from LDS in child order, and then a thread per parent
// solves the 3x3 eigenproblem by cyclic Jacobi rotations (quadratic
// convergence; a sweep limit of 12 is never reached).  It also writes the
// children's parent index and the nodes' child counts.
//
// SH: one thread per float4 (or float) of a parent's SH row, coalesced over
// consecutive parents; this is what bounds the large levels (two million
// leaves of degree 3: 432 MB of SH rows and 103 MB of the rest, 114 us at the
// rate of a copy).
//
// Two million leaves, seven levels of branching 8: 318 us with a thread per
// parent, whose serial loads of eight children (113 us alone) the SH rows of a
// launch of their own (87 us) did not cover; 170 us now.  The upper levels take
// 7 to 12 us each, the latency of one eigenproblem.  Two chunks of children to
// a geometry workgroup (64 parents) rather than one or four (more LDS: fewer
// waves for the SH rows): 180, 218 and 222 us, measured before the period was
// made odd; geometry workgroups dealt in turn rather than first: 180 and 193 us.
// ---------------------------------------------------------------------------
constexpr double kMergeMinVar = 1e-12;

__device__ inline void quat_to_rot_d(double w, double x, double y, double z, double R[9]) {
    const double in = 1.0 / sqrt(w * w + x * x + y * y + z * z);
    w *= in, x *= in, y *= in, z *= in;
    R[0] = 1 - 2 * (y * y + z * z), R[1] = 2 * (x * y - w * z), R[2] = 2 * (x * z + w * y);
    R[3] = 2 * (x * y + w * z), R[4] = 1 - 2 * (x * x + z * z), R[5] = 2 * (y * z - w * x);
    R[6] = 2 * (x * z - w * y), R[7] = 2 * (y * z + w * x), R[8] = 1 - 2 * (x * x + y * y);
}

// Symmetric 3x3 eigendecomposition, a (row-major) overwritten; eigenvalues in
// lam (ascending), eigenvectors in the columns of V (determinant +1).
__device__ inline void sym3_eig(double a[9], double lam[3], double V[9]) {
    for (int i = 0; i < 9; ++i) V[i] = (i % 4 == 0) ? 1.0 : 0.0;
    for (int sweep = 0; sweep < 12; ++sweep) {
        const double off = a[1] * a[1] + a[2] * a[2] + a[5] * a[5];
        const double dia = a[0] * a[0] + a[4] * a[4] + a[8] * a[8];
        if (!(off > 1e-34 * dia)) break;
#pragma unroll
        for (int r = 0; r < 3; ++r) {
            const int p = r == 2 ? 1 : 0, q = r == 0 ? 1 : 2;
            const double apq = a[3 * p + q];
            if (apq == 0.0) continue;
            // tan of the rotation: the smaller root of t^2 + 2 theta t - 1 with theta = d / h
            // (any t gives a rotation; where the squares underflow it is a smaller one)
            const double d = a[3 * q + q] - a[3 * p + p], h = 2.0 * apq;
            const double root = fmax(sqrt(d * d + h * h), fabs(h));
            const double t = h / (d >= 0.0 ? d + root : d - root);
            const double c = 1.0 / sqrt(t * t + 1.0), s = t * c;
            // A <- J^T A J with J the rotation in the (p, q) plane
            for (int k = 0; k < 3; ++k) {  // columns p, q
                const double akp = a[3 * k + p], akq = a[3 * k + q];
                a[3 * k + p] = c * akp - s * akq;
                a[3 * k + q] = s * akp + c * akq;
            }
            for (int k = 0; k < 3; ++k) {  // rows p, q
                const double apk = a[3 * p + k], aqk = a[3 * q + k];
                a[3 * p + k] = c * apk - s * aqk;
                a[3 * q + k] = s * apk + c * aqk;
            }
            a[3 * p + q] = a[3 * q + p] = 0.0;
            for (int k = 0; k < 3; ++k) {  // V <- V J
                const double vkp = V[3 * k + p], vkq = V[3 * k + q];
                V[3 * k + p] = c * vkp - s * vkq;
                V[3 * k + q] = s * vkp + c * vkq;
            }
        }
    }
    lam[0] = a[0], lam[1] = a[4], lam[2] = a[8];
    // ascending, columns along
    for (int i = 0; i < 2; ++i)
        for (int j = 0; j < 2 - i; ++j)
            if (lam[j] > lam[j + 1]) {
                const double tl = lam[j];
                lam[j] = lam[j + 1], lam[j + 1] = tl;
                for (int k = 0; k < 3; ++k) {
                    const double tv = V[3 * k + j];
                    V[3 * k + j] = V[3 * k + j + 1], V[3 * k + j + 1] = tv;
                }
            }
    const double det = V[0] * (V[4] * V[8] - V[5] * V[7]) - V[1] * (V[3] * V[8] - V[5] * V[6]) +
                       V[2] * (V[3] * V[7] - V[4] * V[6]);
    if (det < 0.0)
        for (int k = 0; k < 3; ++k) V[3 * k + 2] = -V[3 * k + 2];
}

// Unit quaternion (w, x, y, z), w >= 0, of a proper rotation matrix: the
// largest of the four squared components is taken from the diagonal, the
// others from sums and differences of the off-diagonal entries over it.
__device__ inline void rot_to_quat_d(const double R[9], double q[4]) {
    const double tr = R[0] + R[4] + R[8];
    const double sq[4] = {1.0 + tr, 1.0 + 2.0 * R[0] - tr, 1.0 + 2.0 * R[4] - tr, 1.0 + 2.0 * R[8] - tr};
    int k = 0;
    for (int i = 1; i < 4; ++i)
        if (sq[i] > sq[k]) k = i;
    const double s = sqrt(fmax(sq[k], 1e-300));  // 2 |q_k|
    const double d = 2.0 * s;
    if (k == 0) {
        q[0] = s / 2, q[1] = (R[7] - R[5]) / d, q[2] = (R[2] - R[6]) / d, q[3] = (R[3] - R[1]) / d;
    } else if (k == 1) {
        q[0] = (R[7] - R[5]) / d, q[1] = s / 2, q[2] = (R[1] + R[3]) / d, q[3] = (R[2] + R[6]) / d;
    } else if (k == 2) {
        q[0] = (R[2] - R[6]) / d, q[1] = (R[1] + R[3]) / d, q[2] = s / 2, q[3] = (R[5] + R[7]) / d;
    } else {
        q[0] = (R[3] - R[1]) / d, q[1] = (R[2] + R[6]) / d, q[2] = (R[5] + R[7]) / d, q[3] = s / 2;
    }
    const double sg = q[0] < 0.0 ? -1.0 : 1.0;
    const double n = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    for (int i = 0; i < 4; ++i) q[i] *= sg / n;
}

constexpr uint32_t kMergeThreads = 256, kMergeMaxParents = 64, kMergeTerms = 11;

struct MergeLevel {
    gsr_param_set nodes;
    uint64_t child_base, n_child, parent_base, n_parent;
    uint32_t branching, per, chunks;  // parents per 256 children; such chunks per geometry workgroup
    uint32_t geometry, period;        // geometry workgroups; every period-th workgroup is one
    bool leaves, roots;               // the children are leaves; the parents are roots
    int32_t *parent, *child_count;
};

// Parent j of the level from its eleven sums.
__device__ __forceinline__ void merge_parent(const MergeLevel &L, uint64_t j, const double *S) {
    const gsr_param_set &nodes = L.nodes;
    const uint64_t b = L.branching, p = L.parent_base + j, c0 = L.child_base + j * b;
    L.child_count[p] = (int32_t)min((uint64_t)b, L.n_child - j * b);
    if (L.roots) L.parent[p] = -1;
    const double inv = 1.0 / S[0];
    const double m[3] = {S[1] * inv, S[2] * inv, S[3] * inv};  // mean about the first child
    double A[9];
    A[0] = S[4] * inv - m[0] * m[0], A[1] = A[3] = S[5] * inv - m[0] * m[1], A[2] = A[6] = S[6] * inv - m[0] * m[2];
    A[4] = S[7] * inv - m[1] * m[1], A[5] = A[7] = S[8] * inv - m[1] * m[2], A[8] = S[9] * inv - m[2] * m[2];
    double lam[3], V[9], q[4];
    sym3_eig(A, lam, V);
    rot_to_quat_d(V, q);
    for (int a = 0; a < 3; ++a) {
        nodes.means[3 * p + a] = (float)((double)nodes.means[3 * c0 + a] + m[a]);
        nodes.log_scales[3 * p + a] = (float)(0.5 * log(fmax(lam[a], kMergeMinVar)));
    }
    reinterpret_cast<float4 *>(nodes.quats)[p] = make_float4((float)q[0], (float)q[1], (float)q[2], (float)q[3]);
    nodes.opacities[p] = (float)(1.0 - S[10]);
}

// Geometry workgroup wg: parents [wg * chunks * per, + chunks * per).
__device__ __forceinline__ void merge_geometry(const MergeLevel &L, uint64_t wg, double (*child)[kMergeTerms],
                                               double (*sums)[kMergeTerms]) {
    const gsr_param_set &nodes = L.nodes;
    const uint32_t tid = threadIdx.x, b = L.branching;
    const uint64_t j0 = wg * L.chunks * L.per;  // the first parent
    const uint32_t np = (uint32_t)min((uint64_t)(L.chunks * L.per), L.n_parent - j0);
    for (uint32_t q0 = 0; q0 < np; q0 += L.per) {
        const uint32_t q = q0 + tid / b;  // the child's parent within the workgroup
        const uint64_t in = (j0 + q0) * b + tid;
        if (tid < L.per * b && q < np && in < L.n_child) {
            const uint64_t c = L.child_base + in, c0 = L.child_base + (j0 + q) * b;
            L.parent[c] = (int32_t)(L.parent_base + j0 + q);
            if (L.leaves) L.child_count[c] = 0;
            const double o = nodes.opacities[c];
            const float4 qf = reinterpret_cast<const float4 *>(nodes.quats)[c];
            double R[9];
            quat_to_rot_d(qf.x, qf.y, qf.z, qf.w, R);
            const double e0 = exp(2.0 * (double)nodes.log_scales[3 * c]),
                         e1 = exp(2.0 * (double)nodes.log_scales[3 * c + 1]),
                         e2 = exp(2.0 * (double)nodes.log_scales[3 * c + 2]);
            const double d[3] = {(double)nodes.means[3 * c] - (double)nodes.means[3 * c0],
                                 (double)nodes.means[3 * c + 1] - (double)nodes.means[3 * c0 + 1],
                                 (double)nodes.means[3 * c + 2] - (double)nodes.means[3 * c0 + 2]};
            double *t = child[tid];
            t[0] = o;
#pragma unroll
            for (int a = 0; a < 3; ++a) t[1 + a] = o * d[a];
            // o (Sigma_c + d d^T), upper triangle: 00 01 02 11 12 22
#pragma unroll
            for (int a = 0, e = 4; a < 3; ++a)
#pragma unroll
                for (int k = a; k < 3; ++k, ++e)
                    t[e] = o * (R[3 * a] * R[3 * k] * e0 + R[3 * a + 1] * R[3 * k + 1] * e1 +
                                R[3 * a + 2] * R[3 * k + 2] * e2 + d[a] * d[k]);
            t[10] = 1.0 - o;
        }
        __syncthreads();
        const uint32_t nq = min(L.per, np - q0);
        for (uint32_t e = tid; e < nq * kMergeTerms; e += kMergeThreads) {
            const uint32_t r = e / kMergeTerms, t = e - r * kMergeTerms;
            const uint32_t k = (uint32_t)min((uint64_t)b, L.n_child - (j0 + q0 + r) * b);
            double x = child[r * b][t];
            if (t < 10)
                for (uint32_t i = 1; i < k; ++i) x += child[r * b + i][t];
            else
                for (uint32_t i = 1; i < k; ++i) x *= child[r * b + i][t];
            sums[q0 + r][t] = x;
        }
        __syncthreads();
    }
    if (tid < np) merge_parent(L, j0 + tid, sums[tid]);
}

// Parent j by a thread of its own, its children one after the other.
__global__ __launch_bounds__(kMergeThreads) void k_merge_serial(MergeLevel L) {
    const uint64_t j = (uint64_t)blockIdx.x * kMergeThreads + threadIdx.x;
    if (j >= L.n_parent) return;
    const gsr_param_set &nodes = L.nodes;
    const uint64_t first = j * L.branching, c0 = L.child_base + first;
    const uint32_t k = (uint32_t)min((uint64_t)L.branching, L.n_child - first);
    const double ox = nodes.means[3 * c0], oy = nodes.means[3 * c0 + 1], oz = nodes.means[3 * c0 + 2];
    double S[kMergeTerms] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 1.0};
    for (uint32_t i = 0; i < k; ++i) {
        const uint64_t c = c0 + i;
        L.parent[c] = (int32_t)(L.parent_base + j);
        if (L.leaves) L.child_count[c] = 0;
        const double o = nodes.opacities[c];
        const float4 qf = reinterpret_cast<const float4 *>(nodes.quats)[c];
        double R[9];
        quat_to_rot_d(qf.x, qf.y, qf.z, qf.w, R);
        const double e0 = exp(2.0 * (double)nodes.log_scales[3 * c]), e1 = exp(2.0 * (double)nodes.log_scales[3 * c + 1]),
                     e2 = exp(2.0 * (double)nodes.log_scales[3 * c + 2]);
        const double d[3] = {(double)nodes.means[3 * c] - ox, (double)nodes.means[3 * c + 1] - oy,
                             (double)nodes.means[3 * c + 2] - oz};
        S[0] += o;
#pragma unroll
        for (int a = 0; a < 3; ++a) S[1 + a] += o * d[a];
#pragma unroll
        for (int a = 0, e = 4; a < 3; ++a)
#pragma unroll
            for (int q = a; q < 3; ++q, ++e)
                S[e] += o * (R[3 * a] * R[3 * q] * e0 + R[3 * a + 1] * R[3 * q + 1] * e1 +
                             R[3 * a + 2] * R[3 * q + 2] * e2 + d[a] * d[q]);
        S[10] *= 1.0 - o;
    }
    merge_parent(L, j, S);
}

// Unit t of the parents' SH rows (K3 / 4 float4 units a row, or K3 floats when
// a row is not a whole number of float4).
template <int K3, bool VEC, int UNROLL>
__device__ __forceinline__ void merge_sh(const MergeLevel &L, uint64_t t) {
    constexpr uint32_t kUnits = VEC ? K3 / 4 : K3;
    const gsr_param_set &nodes = L.nodes;
    if (t >= L.n_parent * kUnits) return;
    const uint64_t j = t / kUnits, u = t - j * kUnits;
    const uint64_t first = j * L.branching, c0 = L.child_base + first, p = L.parent_base + j;
    const uint32_t k = (uint32_t)min((uint64_t)L.branching, L.n_child - first);
    float wsum = 0.f;
#pragma unroll UNROLL
    for (uint32_t i = 0; i < k; ++i) wsum += nodes.opacities[c0 + i];
    const float inv = 1.f / wsum;
    if constexpr (VEC) {
        float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll UNROLL
        for (uint32_t i = 0; i < k; ++i) {
            const float w = nodes.opacities[c0 + i] * inv;
            const float4 v = reinterpret_cast<const float4 *>(nodes.sh)[(c0 + i) * kUnits + u];
            acc.x = fmaf(w, v.x, acc.x), acc.y = fmaf(w, v.y, acc.y), acc.z = fmaf(w, v.z, acc.z),
            acc.w = fmaf(w, v.w, acc.w);
        }
        reinterpret_cast<float4 *>(nodes.sh)[p * kUnits + u] = acc;
    } else {
        float acc = 0.f;
#pragma unroll UNROLL
        for (uint32_t i = 0; i < k; ++i) acc = fmaf(nodes.opacities[c0 + i] * inv, nodes.sh[(c0 + i) * kUnits + u], acc);
        nodes.sh[p * kUnits + u] = acc;
    }
}

template <int K3, bool VEC>
__global__ __launch_bounds__(kMergeThreads, 4) void k_merge_level(MergeLevel L) {
    __shared__ double child[kMergeThreads][kMergeTerms], sums[kMergeMaxParents][kMergeTerms];
    const uint32_t turn = blockIdx.x / L.period;
    if (turn * L.period == blockIdx.x && turn < L.geometry) {  // uniform
        merge_geometry(L, turn, child, sums);
        return;
    }
    // the SH workgroups are those between, numbered through
    const uint64_t wg = blockIdx.x - min(L.geometry, turn + 1);
    merge_sh<K3, VEC, 8>(L, wg * kMergeThreads + threadIdx.x);
}

template <int K3, bool VEC>
__global__ __launch_bounds__(kMergeThreads) void k_merge_sh(MergeLevel L) {
    merge_sh<K3, VEC, 4>(L, (uint64_t)blockIdx.x * kMergeThreads + threadIdx.x);
}

__global__ __launch_bounds__(256) void k_fill_i32(int32_t *__restrict__ p, int32_t value, uint64_t n) {
    const uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < n) p[i] = value;
}

// Parents of a launch: at most 2^32 threads are launched at a time, of up to 27 a
// parent for the SH rows and 4 or so for the geometry.
constexpr uint64_t kMergeMaxLaunch = 1ull << 26;

static void launch_level_part(const gsr_param_set &nodes, int sh_degree, uint64_t child_base, uint64_t n_child,
                              uint64_t parent_base, uint32_t branching, bool leaves, bool roots, int32_t *parent,
                              int32_t *child_count, hipStream_t st) {
    MergeLevel L{};
    L.nodes = nodes;
    L.child_base = child_base, L.n_child = n_child, L.parent_base = parent_base;
    L.n_parent = (n_child + branching - 1) / branching;
    L.branching = branching;
    L.per = std::min(kMergeThreads / branching, kMergeMaxParents);
    // two chunks to a workgroup, so that the parents' part runs on a full wave,
    // once that leaves four workgroups per compute unit
    L.chunks = (uint32_t)std::max<uint64_t>(
        1, std::min<uint64_t>(kMergeMaxParents / L.per, L.n_parent / (L.per * 1024ull)));
    L.geometry = (uint32_t)((L.n_parent + L.per * L.chunks - 1) / (L.per * L.chunks));
    L.leaves = leaves, L.roots = roots;
    L.parent = parent, L.child_count = child_count;
    // Large levels of few children a parent: the SH rows in a launch of their own, where
    // no LDS keeps waves away, and up to five children the geometry by a thread per
    // parent (64 threads of a workgroup would have a parent, and few a child).  One
    // launch / apart, us: 1 M parents of three 160 / 121, 181 / 147, 419 / 268 and 319 / 239
    // (degrees 0 to 3); 1.6 M of five 513 / 484 (degree 0, with the levels above); 500 k of
    // six 358 / 232 and 270 / 251 (2 and 3); 375 k of eight 167 / 215 (3); 66 k of three 17.2 /
    // 19.9, 34.5 / 28.1 and 27.1 / 26.8 (0, 2 and 3); 33 k of six 28.9 / 25.6 and 17.0 / 23.9 (2 and 3).
    const bool rows = sh_degree >= 2, serial = branching <= 5;
    const bool apart = branching <= (rows ? 7u : L.n_parent >= 1ull << 20 ? 5u : 4u) &&
                       L.n_parent >= (sh_degree == 2 || (rows && serial) ? 1ull << 15 : 1ull << 18);
    auto run = [&](auto level, auto sh_rows, uint64_t units) {
        const uint32_t sh = (uint32_t)((L.n_parent * units + kMergeThreads - 1) / kMergeThreads);
        if (!apart) {
            // an odd period: workgroups go to the XCDs and their shader engines in turn, and an
            // even one gives the geometry to some of them only (8 M leaves of degree 3,
            // branching 8: 1,036 us with a period of 4, 556 us with 3)
            L.period = (L.geometry + sh) / L.geometry;
            if (L.period % 2 == 0) --L.period;
            hipLaunchKernelGGL(level, dim3(L.geometry + sh), dim3(kMergeThreads), 0, st, L);
            return;
        }
        L.period = 1;
        if (serial)
            hipLaunchKernelGGL(k_merge_serial, dim3((unsigned)((L.n_parent + kMergeThreads - 1) / kMergeThreads)),
                               dim3(kMergeThreads), 0, st, L);
        else
            hipLaunchKernelGGL(level, dim3(L.geometry), dim3(kMergeThreads), 0, st, L);
        hipLaunchKernelGGL(sh_rows, dim3(sh), dim3(kMergeThreads), 0, st, L);
    };
    switch (sh_degree) {
        case 0: run(k_merge_level<3, false>, k_merge_sh<3, false>, 3); break;
        case 1: run(k_merge_level<12, true>, k_merge_sh<12, true>, 3); break;
        case 2: run(k_merge_level<27, false>, k_merge_sh<27, false>, 27); break;
        default: run(k_merge_level<48, true>, k_merge_sh<48, true>, 12); break;
    }
}

void launch_hierarchy_level(const gsr_param_set &nodes, int sh_degree, uint64_t child_base, uint64_t n_child,
                            uint64_t parent_base, uint32_t branching, bool leaves, bool roots, int32_t *parent,
                            int32_t *child_count, hipStream_t st) {
    const uint64_t step = kMergeMaxLaunch * branching;  // whole parents
    for (uint64_t c = 0; c < n_child; c += step)
        launch_level_part(nodes, sh_degree, child_base + c, std::min(step, n_child - c), parent_base + c / branching,
                          branching, leaves, roots, parent, child_count, st);
}

void launch_fill_i32(int32_t *p, int32_t value, uint64_t n, hipStream_t st) {
    if (n == 0) return;
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, p, value, n);
}

}  // namespace gsr
