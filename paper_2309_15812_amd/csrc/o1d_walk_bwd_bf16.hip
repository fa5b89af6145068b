// Walk kernels: both gradients in one pass, bf16 storage, nchw.
#include "o1d_walk_kernels.h"

namespace o1d {

hipError_t launch_walk_bwd_bf16(const walk::Plan& pl, const void* x, const void* dy, const void* w, const float* theta,
                               void* dx, float* partial, hipStream_t stream) {
  return walk::bwd_t<uint16_t>(pl, x, dy, w, theta, dx, partial, stream);
}

}  // namespace o1d
