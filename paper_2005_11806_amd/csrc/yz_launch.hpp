// y pass kernels and their dispatch over lengths and chunk rows, instantiated
// once per precision (kernels_yz.hip FP64, kernels_yz32.hip FP32).
#pragma once

#include "jobs.hpp"
#include "pass_yz.hpp"

namespace psv {

void launch_yz64(const Plan& p, const ZArgs& z, bool inverse, const Job& job, const int* done,
                 hipStream_t s);
void launch_yz32(const Plan& p, const ZArgs& z, bool inverse, const Job& job, const int* done,
                 hipStream_t s);

namespace {

constexpr int JOB_BLOCKS = 8;

template <typename T, int N, int KC, bool INV>
__global__ void __launch_bounds__(N ? yz_threads(N, KC) : 256) k_yz(ZArgs z, Radices rad, c2<T>* __restrict__ spec,
                                            const c2<T>* __restrict__ tw_g, const int* done, Job job) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (done && *done) return;
    int b = blockIdx.x;
    if constexpr (!INV) {
        // block 0 takes the job, if there is one. Eight blocks go before the tiles
        // then, which keeps each tile on the XCD it has in the inverse pass: with
        // one, that pass found its rows in another L2 (128^3: 13.5 us against 8.3).
        if (job.kind != JOB_NONE && (b -= JOB_BLOCKS) < 0) {
            if (blockIdx.x == 0) run_job(job, reinterpret_cast<double*>(smem_raw));
            return;
        }
    }
    if constexpr (INV)
        yz_inv_tile<T, N, KC, yz_threads(N, KC)>(z, rad, spec, tw_g, b, smem_raw);
    else
        yz_fwd_tile<T, N, KC, yz_threads(N, KC)>(z, rad, spec, tw_g, b, smem_raw);
}

// Two-dimensional problems (ny = 1): the y transform is the identity and a y
// tile would hold a single system, so here one thread takes the chunk of one
// wavenumber m (consecutive threads, consecutive m: the rows of a plane are
// read and written whole). Same arithmetic as the tiles: the forward chunk is
// eliminated in registers (rows past nz read as 0), the inverse one
// back-substituted in place.
template <typename T, int KC, bool INV>
__global__ void __launch_bounds__(256) k_z2d(ZArgs z, c2<T>* __restrict__ spec, const int* done, Job job) {
    __shared__ double sh[16];
    if (done && *done) return;
    if constexpr (!INV) {  // the row of blocks past the chunks: block 0 takes the job
        if ((int)blockIdx.y == z.nc) {
            if (blockIdx.x == 0) run_job(job, sh);
            return;
        }
    }
    const int m = (int)blockIdx.x * 256 + (int)threadIdx.x;
    if (m == 0 || m >= z.mx) return;  // the (0,0) pair is solved apart
    const int k0 = (int)blockIdx.y * KC;
    const int nl = min(KC, z.nz - k0);
    const int SP = z.mx;  // elements per plane when ny = 1
    c2<T>* col = spec + (size_t)k0 * SP + m;
    const double lam = z.lamx[m] + z.lamy[0];
    c2<T> v[KC];
#pragma unroll
    for (int i = 0; i < KC; ++i) v[i] = i < nl ? col[(size_t)i * SP] : c2<T>{(T)0, (T)0};
    if constexpr (INV)
        chunk_substitute<T, KC>(zrows(z, k0, lam), nl, v);
    else
        chunk_eliminate<T, KC>(zrows(z, k0, lam), v);
#pragma unroll
    for (int i = 0; i < KC; ++i)
        if (i < nl) col[(size_t)i * SP] = v[i];
}

template <typename T, bool INV>
void z2d_launch(const Plan& p, const ZArgs& z, c2<T>* spec, const Job& job, const int* done, hipStream_t s) {
    const dim3 grid((p.mx + 255) / 256, z.nc + (!INV && job.kind != JOB_NONE ? 1 : 0));
    switch (p.lp.kc) {
        case 4: hipLaunchKernelGGL((k_z2d<T, 4, INV>), grid, dim3(256), 0, s, z, spec, done, job); break;
        case 8: hipLaunchKernelGGL((k_z2d<T, 8, INV>), grid, dim3(256), 0, s, z, spec, done, job); break;
        default: hipLaunchKernelGGL((k_z2d<T, 16, INV>), grid, dim3(256), 0, s, z, spec, done, job); break;
    }
}

template <typename T, int N, int KC, bool INV>
void yz_launch(const Plan& p, const ZArgs& z, c2<T>* spec, const c2<T>* tw, const Job& job,
               const int* done, hipStream_t s) {
    const size_t lds = yz_lds(p.ny, KC, sizeof(c2<T>), N > 0);
    allow_lds(k_yz<T, N, KC, INV>, lds);
    hipLaunchKernelGGL((k_yz<T, N, KC, INV>), dim3(yz_tiles(p) + (!INV && job.kind != JOB_NONE ? JOB_BLOCKS : 0)), dim3(yz_threads(N, KC)), lds, s, z,
                       p.rad_y,
                       spec, tw, done, job);
}

template <typename T, int N, bool INV>
void yz_dispatch_kc(const Plan& p, const ZArgs& z, c2<T>* spec, const c2<T>* tw, const Job& job,
                    const int* done, hipStream_t s) {
    switch (p.lp.kc) {
        case 4: yz_launch<T, N, 4, INV>(p, z, spec, tw, job, done, s); break;
        case 8: yz_launch<T, N, 8, INV>(p, z, spec, tw, job, done, s); break;
        default: yz_launch<T, N, 16, INV>(p, z, spec, tw, job, done, s); break;
    }
}

template <typename T, bool INV>
void yz_dispatch(const Plan& p, const ZArgs& z, c2<T>* spec, const c2<T>* tw, const Job& job,
                 const int* done, hipStream_t s) {
    if (p.ny == 1) {
        z2d_launch<T, INV>(p, z, spec, job, done, s);
        return;
    }
    switch (p.ny) {
#define PSV_CASE(n) case n: yz_dispatch_kc<T, n, INV>(p, z, spec, tw, job, done, s); break;
        PSV_YZ_SIZES(PSV_CASE)
        PSV_YZ_MORE(PSV_CASE)
#undef PSV_CASE
        default: yz_dispatch_kc<T, 0, INV>(p, z, spec, tw, job, done, s); break;
    }
}

}  // namespace
}  // namespace psv
