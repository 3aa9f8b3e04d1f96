// gsr_ba.h -- device-side interface of the local bundle adjustment (FP64):
// sizes, the argument block its kernels share, and the launchers.
#pragma once
#include "gsr_internal.h"

namespace gsr {

// ---- local bundle adjustment (FP64) ----
constexpr int kBaMaxObs = 8;       // observation slots per landmark (lanes per landmark)
constexpr int kBaMaxFree = 20;     // free keyframes: reduced system of 6 * 20 + 1 unknowns
constexpr int kBaLmStride = 16;    // doubles per landmark record (15 used): one cache line
constexpr int kBaAsmSplit = 2;     // workgroups (partial systems) per block of the reduced system

struct BaArgs {
    double *poses, *focal, *landmarks;
    const double *obs_uv;
    const int32_t *obs_cam, *free_slot, *slot_cam;
    const int2 *block_ab;
    // per block of the reduced system, in landmark order: a diagonal block's
    // observations (landmark * M + slot), an off-diagonal one's shared landmarks
    const uint32_t *pairs, *block_off;
    double *lm_rec, *lm_sum;   // per landmark; per block of the landmark pass: 4 sums
    double *S, *dc, *costs;
    double *pose_old;          // [F][12] free poses before the last step, then the focal length before it
    double cx, cy, lambda;
    int K, M, F, D, nblk;
};

size_t ba_lds_bytes(int D);        // largest dynamic LDS of the solver's kernels
hipError_t ba_allow_lds(int D);
size_t ba_lm_blocks(int K);        // workgroups of the landmark pass
void launch_ba_iterations(const BaArgs &A, int iterations, hipStream_t st);

}  // namespace gsr
