// Forward and inverse x passes: FP32 kernels.
#include "x_launch.hpp"

namespace psv {

void launch_fwd_x32(const Plan& p, const FwdArgs& a, hipStream_t s) { fwd_modes<float>(p, a, s); }

void launch_inv_x32(const Plan& p, int mode, double* out, double scale_all, const int* done,
                    hipStream_t s, int max_blocks) {
    inv_modes<float>(p, mode, out, scale_all, done, s, max_blocks);
}

}  // namespace psv
