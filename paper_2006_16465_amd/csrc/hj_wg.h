// hj_wg.h -- what the one-workgroup solves share: the verdict's running state,
// the sum of a cycle's wavefront sums and the opt-in to large LDS.
#pragma once

#include "hj_device.h"

namespace hj {
namespace {

// Dynamic LDS above the default 64 KiB needs the kernel's opt-in.
template <typename K>
hipError_t allow_lds(K kernel, size_t lds)
{
    if (lds <= 64 * 1024) return hipSuccess;
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
}

// Sum of the wavefront sums of one cycle: a fixed tree over SL slots (slots
// of wavefronts the workgroup does not have hold 0, so SL = 8 and SL = 16 add
// the same numbers in the same order).
template <int SL>
__device__ __forceinline__ double tree_sum(const double *slot)
{
    double p[SL];
#pragma unroll
    for (int w = 0; w < SL; ++w) p[w] = slot[w];
#pragma unroll
    for (int h = SL / 2; h >= 1; h >>= 1)
#pragma unroll
        for (int w = 0; w < h; ++w) p[w] += p[w + h];
    return p[0];
}

// The verdict's running state, identical in every thread.
struct WgJudge {
    double r0sq, last, lim, tol;
    int64_t done;
    int32_t status;

    // Limit above which a sum cannot meet the tolerance: the exact verdict
    // rel = sqrt(tot) / sqrt(r0sq) <= tol is skipped while tot exceeds
    // tol^2 r0sq by a margin (1e-6) far above the rounding of either form.
    // Only a normal bound is trusted (no underflow), and none before the
    // first residual: inf sends a cycle through the exact form.
    __device__ __forceinline__ void set_lim()
    {
        const double bound = tol * tol * r0sq * (1.0 + 1e-6);
        lim = bound >= 0x1p-1000 && bound <= 0x1p1000 ? bound : INFINITY;
    }

    __device__ __forceinline__ bool far(double tot) const { return tot > lim && tot < INFINITY; }

    // the exact verdict on iterate c
    __device__ __forceinline__ void take(int64_t c, double tot)
    {
        if (status != ST_RUNNING) return;
        last = tot;
        if (c == 0) {
            r0sq = tot;
            set_lim();
        }
        if (!isfinite(tot)) {
            status = ST_NONFINITE;
        } else {
            const double rel = r0sq > 0.0 ? sqrt(tot) / sqrt(r0sq) : 0.0;
            if (rel <= tol) status = ST_CONVERGED;
        }
        if (status != ST_RUNNING) done = c;
    }
};

}  // namespace
}  // namespace hj
