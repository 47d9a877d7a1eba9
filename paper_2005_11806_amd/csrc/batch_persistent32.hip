// Persistent batched executor, FP32.
#include "batch_persistent.hpp"

namespace psv {

void launch_queue32(const PersistArgs& A, size_t lds, int device, hipStream_t s) {
    launch_queue<float>(A, lds, device, s);
}

}  // namespace psv
