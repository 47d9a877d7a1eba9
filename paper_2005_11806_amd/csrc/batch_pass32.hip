// Per-pass batched kernels, FP32.
#include "batch_pass.hpp"

namespace psv {

void launch_pass32(const PassLaunch& L, const ProblemDesc* desc, const ProblemIO* io, int n, hipStream_t s) {
    launch_pass<float>(L, desc, io, n, s);
}

}  // namespace psv
