// Single-block jobs on the partial sums of a forward x pass (Job in
// internal.hpp), run by a block of their own or by an extra block of the
// forward y pass.
#pragma once

#include "internal.hpp"

namespace psv {

// This thread's share (threads 0..255) of the sum of every `stride`-th of the nb
// entries of p, in a fixed order. Four loads in flight and one sum at a time: the
// kernels that carry the jobs need no more registers than without them.
__device__ __forceinline__ double job_share(const double* p, int nb, int stride) {
    double a0 = 0.0, a1 = 0.0, a2 = 0.0, a3 = 0.0;
    unsigned b = threadIdx.x;
    if (b >= 256) return 0.0;
#pragma unroll 1
    for (; b + 768 < (unsigned)nb; b += 1024) {
        const double v0 = at_off(p, b * stride), v1 = at_off(p, (b + 256) * stride),
                     v2 = at_off(p, (b + 512) * stride), v3 = at_off(p, (b + 768) * stride);
        a0 += v0;
        a1 += v1;
        a2 += v2;
        a3 += v3;
    }
#pragma unroll 1
    for (; b < (unsigned)nb; b += 256) a0 += at_off(p, b * stride);
    return (a0 + a1) + (a2 + a3);
}

// The whole block takes part (256 or 512 threads); sh: 16 doubles of LDS.
__device__ __forceinline__ void run_job(const Job& j, double* sh) {
    double* scal = j.scal;
    int* flags = j.flags;
    if (j.kind != JOB_MEAN && flags[F_DONE]) return;  // uniform over the block
    const int per = j.kind == JOB_REFINE ? 2 : 1;
    const double t = block_sum(job_share(j.partials, j.nb, per), sh);
    if (j.kind == JOB_REFINE) {
        __syncthreads();
        const double a = t, b = block_sum(job_share(j.partials + 1, j.nb, 2), sh);
        if (threadIdx.x != 0) return;
        const double rr = b > 0.0 ? sqrt(a / b) : 0.0;
        // The residual left by the FP32 solve is rounding at the grid's scale, which a
        // correction takes down by 2.3e-7 to 4.8e-7 (16 grids, uniform and stretched,
        // three two-phase inputs each; 6e-7 to 1e-6 with chunk rows other than the
        // built-in ones, the more for noise). The upper end: a residual wrongly expected to be the last costs a
        // whole further pass, 125 us at 256 x 256 x 512, one not expected to be 47 us.
        flags[F_REDO] = flags[F_LAST];
        flags[F_LAST] = 5e-7 * rr <= j.tol;
        scal[S_RELRES] = rr;
        if (j.sweep < S_NHIST) scal[S_HIST + j.sweep] = rr;
        if (rr <= j.tol) {
            flags[F_DONE] = 1;
            flags[F_CONV] = 1;
        } else if (j.sweep >= j.max_iter || !isfinite(rr)) {
            flags[F_DONE] = 1;
        } else {
            flags[F_STEPS] += 1;
        }
        return;
    }
    if (j.kind == JOB_MEAN) {
        if (threadIdx.x < S_NHIST) scal[S_HIST + threadIdx.x] = __builtin_nan("");
        if (threadIdx.x != 0) return;
        scal[S_RHS_MEAN] = t / j.total;
        flags[F_DONE] = 0;
        flags[F_GATE] = 0;
        flags[F_LAST] = 0;
        flags[F_REDO] = 0;
        flags[F_STEPS] = 0;
        flags[F_CONV] = 0;
        return;
    }
    if (threadIdx.x != 0) return;
    const double eps = j.total * t;
    scal[S_HIST + (flags[F_STEPS] & 7)] = eps;  // after F_STEPS solves
    if (!j.has_p) {
        scal[S_EPS0] = eps;
    } else {
        scal[S_EPS] = eps;
        if (eps <= j.tol) {
            flags[F_CONV] = 1;
            flags[F_DONE] = 1;
            return;
        }
        if (flags[F_STEPS] >= j.max_iter) {
            flags[F_DONE] = 1;
            return;
        }
    }
    flags[F_STEPS] += 1;
}

}  // namespace psv
