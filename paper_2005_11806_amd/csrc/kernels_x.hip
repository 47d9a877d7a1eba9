// Forward and inverse x passes: FP64 kernels and the entry points.
#include "x_launch.hpp"

namespace psv {

int fwd_x_blocks(const Plan& p) { return (p.ny / p.lp.lbx) * p.nz; }

void launch_fwd_x(const Plan& p, bool fp32, const FwdArgs& a, hipStream_t s) {
    if (fp32)
        launch_fwd_x32(p, a, s);
    else
        fwd_modes<double>(p, a, s);
}

void launch_inv_x(const Plan& p, bool fp32, int mode, double* out, double scale_all,
                  const int* done, hipStream_t s, int max_blocks) {
    if (fp32)
        launch_inv_x32(p, mode, out, scale_all, done, s, max_blocks);
    else
        inv_modes<double>(p, mode, out, scale_all, done, s, max_blocks);
}

}  // namespace psv
