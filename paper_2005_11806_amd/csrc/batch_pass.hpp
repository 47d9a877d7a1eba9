// Per-pass batched kernels of one precision.
#pragma once

#include "batch_tasks.hpp"

namespace psv {
namespace {

// Per-pass batched kernel: block -> (problem, tile) through start[] (prefix of
// tile counts, nprob + 1 entries). SEL: the launch's variant (PassLaunch::sel;
// problems of another variant have no tiles in this launch). The inverse y kernel
// of 8 chunk rows is held to five waves (96 registers; 106 without: 27 million
// cells in 12 problems 450 us against 430).
template <typename T, int KIND, int SEL>
__global__ void __launch_bounds__(256, KIND == K_YI && SEL == 8 ? 5 : 1) k_batch_pass(const ProblemDesc* __restrict__ desc,
                                                     const ProblemIO* __restrict__ io,
                                                     const int* __restrict__ start, int nprob) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ double red[16];
    const int blk = blockIdx.x;
    int lo = 0, hi = nprob;  // largest p with start[p] <= blk
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (start[mid] <= blk) lo = mid; else hi = mid;
    }
    run_task<T, KIND, SEL>(desc[lo], io[lo], blk - start[lo], smem_raw, red);
}

template <typename T, int KIND, int SEL>
void launch_pass_k(const PassLaunch& L, const ProblemDesc* desc, const ProblemIO* io, int n, hipStream_t s) {
    allow_lds(k_batch_pass<T, KIND, SEL>, L.lds);
    hipLaunchKernelGGL((k_batch_pass<T, KIND, SEL>), dim3(L.nblk), dim3(256), L.lds, s, desc, io,
                       L.d_start, n);
}

template <typename T>
void launch_pass(const PassLaunch& L, const ProblemDesc* desc, const ProblemIO* io, int n, hipStream_t s) {
    switch (L.kind) {
#define PSV_K(k) case k: launch_pass_k<T, k, 1>(L, desc, io, n, s); break;
        PSV_K(K_MINP) PSV_K(K_MINF) PSV_K(K_MEAN) PSV_K(K_INV) PSV_K(K_INVADD) PSV_K(K_NRM) PSV_K(K_CHK) PSV_K(K_CHKF)
#undef PSV_K
#define PSV_K(k, a, b, c) case k: \
            if (L.sel == a) launch_pass_k<T, k, a>(L, desc, io, n, s); \
            else if (L.sel == b) launch_pass_k<T, k, b>(L, desc, io, n, s); \
            else launch_pass_k<T, k, c>(L, desc, io, n, s); \
            break;
        PSV_K(K_Y, 4, 8, 16) PSV_K(K_YI, 4, 8, 16) PSV_K(K_Z, 4, 8, 16) PSV_K(K_Z2, 4, 8, 16)
#undef PSV_K
        case K_FWD:
            if (L.sel) launch_pass_k<T, K_FWD, 1>(L, desc, io, n, s); else launch_pass_k<T, K_FWD, 0>(L, desc, io, n, s);
            break;
        case K_RES:
            if (L.sel) launch_pass_k<T, K_RES, 1>(L, desc, io, n, s); else launch_pass_k<T, K_RES, 0>(L, desc, io, n, s);
            break;
    }
    PSV_HIP(hipGetLastError());
}

}  // namespace
}  // namespace psv
