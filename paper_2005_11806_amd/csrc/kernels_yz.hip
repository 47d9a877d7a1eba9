// Per-pass kernels of the y (FP64) and z directions (tile bodies in
// pass_yz.hpp) and the plan-time interface factor table.
#include "yz_launch.hpp"

namespace psv {
namespace {

template <typename T, int QM>
__global__ void __launch_bounds__(IFC_THREADS) k_ifc(ZArgs z, c2<T>* __restrict__ spec, const int* done) {
    extern __shared__ __align__(16) unsigned char smem_raw[];
    if (done && *done) return;
    ifc_tile<T, QM>(z, spec, blockIdx.x, smem_raw);
}

template <typename T, int QM>
void ifc_launch(const Plan& p, const ZArgs& z, const int* done, hipStream_t s) {
    const size_t lds = ifc_lds(p);
    allow_lds(k_ifc<T, QM>, lds);
    hipLaunchKernelGGL((k_ifc<T, QM>), dim3(ifc_tiles(p)), dim3(IFC_THREADS), lds, s, z,
                       reinterpret_cast<c2<T>*>(p.spec), done);
}

template <typename T>
void ifc_dispatch(const Plan& p, const ZArgs& z, const int* done, hipStream_t s) {
    switch (ifc_qmax(2 * z.nc)) {
        case 2: ifc_launch<T, 2>(p, z, done, s); break;
        case 4: ifc_launch<T, 4>(p, z, done, s); break;
        case 8: ifc_launch<T, 8>(p, z, done, s); break;
        default: ifc_launch<T, 16>(p, z, done, s); break;
    }
}

constexpr int TAB_THREADS = 64;

template <typename T, int KC>
__global__ void __launch_bounds__(TAB_THREADS) k_ifc_table(ZArgs z, T* __restrict__ tab) {
    const int s = blockIdx.x * TAB_THREADS + (int)threadIdx.x;
    if (s < z.mx * z.ny) ifc_table_pair<T, KC>(z, s, tab);
}

template <typename T>
void ifc_table_launch(const Plan& p, hipStream_t s) {
    const ZArgs z = make_zargs(p, nullptr);
    const dim3 grid((p.mx * p.ny + TAB_THREADS - 1) / TAB_THREADS), block(TAB_THREADS);
    T* tab = reinterpret_cast<T*>(p.ifc_tab);
    switch (p.lp.kc) {
        case 4: hipLaunchKernelGGL((k_ifc_table<T, 4>), grid, block, 0, s, z, tab); break;
        case 8: hipLaunchKernelGGL((k_ifc_table<T, 8>), grid, block, 0, s, z, tab); break;
        default: hipLaunchKernelGGL((k_ifc_table<T, 16>), grid, block, 0, s, z, tab); break;
    }
}

void check_precision(const Plan& p, bool fp32) {
    if (fp32 != (p.opts.precision == PSV_MIXED))
        fail(PSV_ERR_INVALID_ARG, "z pass precision differs from the plan's");
}

}  // namespace

void launch_yz(const Plan& p, bool fp32, bool inverse, const int* done, hipStream_t s, const Job& job) {
    check_precision(p, fp32);
    static const char* names[2][2] = {{"yz_fwd_fp64", "yz_inv_fp64"}, {"yz_fwd_fp32", "yz_inv_fp32"}};
    TraceScope ts(p, names[fp32][inverse], s);
    const ZArgs z = make_zargs(p, nullptr);
    if (fp32)
        launch_yz32(p, z, inverse, job, done, s);
    else
        launch_yz64(p, z, inverse, job, done, s);
    PSV_HIP(hipGetLastError());
}

void launch_yz64(const Plan& p, const ZArgs& z, bool inverse, const Job& job, const int* done,
                 hipStream_t s) {
    if (inverse)
        yz_dispatch<double, true>(p, z, (double2*)p.spec, p.t.twy64, job, done, s);
    else
        yz_dispatch<double, false>(p, z, (double2*)p.spec, p.t.twy64, job, done, s);
}

void launch_interface(const Plan& p, bool fp32, double* mean_out, const int* done, hipStream_t s) {
    check_precision(p, fp32);
    const ZArgs z = make_zargs(p, mean_out);
    TraceScope ts(p, fp32 ? "z_interface_fp32" : "z_interface_fp64", s);
    if (fp32)
        ifc_dispatch<float>(p, z, done, s);
    else
        ifc_dispatch<double>(p, z, done, s);
    PSV_HIP(hipGetLastError());
}

void launch_z_solve(const Plan& p, bool fp32, double* mean_out, const int* done, hipStream_t s,
                    const Job& job) {
    // see F_GATE
    const int* gate = done && job.kind != JOB_NONE ? done + (F_GATE - F_DONE) : done;
    check_precision(p, fp32);
    if (zf_fits(p)) {
        launch_zf(p, fp32, mean_out, gate, s, job);
        return;
    }
    launch_yz(p, fp32, false, gate, s, job);
    launch_interface(p, fp32, mean_out, done, s);
    launch_yz(p, fp32, true, done, s);
}

bool kc_fits(const Plan& p, int kc) {
    if (kc != 4 && kc != 8 && kc != 16) return false;
    // the batched kernels' tile, which is never the smaller one
    const size_t csz = p.opts.precision == PSV_MIXED ? sizeof(float2) : sizeof(double2);
    return yz_lds(p.ny, kc, csz, yz_batch_compiled(p.ny)) <= (size_t)LDS_MAX_BLOCK;
}

size_t ifc_table_bytes(const Plan& p, int kc) {
    const size_t esz = p.opts.precision == PSV_MIXED ? sizeof(float) : sizeof(double);
    const int nc = (p.nz + kc - 1) / kc;
    return ifc_tab_entries(ifc_shape(nc, p.mx * p.ny)) * esz;
}

void launch_ifc_table(const Plan& p, hipStream_t s) {
    if (p.opts.precision == PSV_MIXED)
        ifc_table_launch<float>(p, s);
    else
        ifc_table_launch<double>(p, s);
    PSV_HIP(hipGetLastError());
}

void plan_set_kc(Plan& p, int kc) {
    if (!kc_fits(p, kc)) fail(PSV_ERR_UNSUPPORTED_SIZE, "chunk rows do not fit the LDS of a block");
    const size_t bytes = ifc_table_bytes(p, kc);
    if (bytes > p.ifc_tab_bytes) {
        if (p.ifc_tab) PSV_HIP(hipFree(p.ifc_tab));
        p.ifc_tab = nullptr;
        p.ifc_tab_bytes = 0;
        PSV_HIP(hipMalloc(&p.ifc_tab, bytes));
        p.ifc_tab_bytes = bytes;
    }
    p.lp.kc = kc;
    launch_ifc_table(p, nullptr);
    PSV_HIP(hipDeviceSynchronize());
}

}  // namespace psv
