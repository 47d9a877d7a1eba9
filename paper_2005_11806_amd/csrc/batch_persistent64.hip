// Persistent batched executor, FP64.
#include "batch_persistent.hpp"

namespace psv {

void launch_queue64(const PersistArgs& A, size_t lds, int device, hipStream_t s) {
    launch_queue<double>(A, lds, device, s);
}

}  // namespace psv
