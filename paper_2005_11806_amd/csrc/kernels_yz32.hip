// FP32 kernels of the y direction.
#include "yz_launch.hpp"

namespace psv {

void launch_yz32(const Plan& p, const ZArgs& z, bool inverse, const Job& job, const int* done,
                 hipStream_t s) {
    if (inverse)
        yz_dispatch<float, true>(p, z, (float2*)p.spec, p.t.twy32, job, done, s);
    else
        yz_dispatch<float, false>(p, z, (float2*)p.spec, p.t.twy32, job, done, s);
}

}  // namespace psv
