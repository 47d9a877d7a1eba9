// Per-pass batched kernels, FP64.
#include "batch_pass.hpp"

namespace psv {

void launch_pass64(const PassLaunch& L, const ProblemDesc* desc, const ProblemIO* io, int n, hipStream_t s) {
    launch_pass<double>(L, desc, io, n, s);
}

}  // namespace psv
