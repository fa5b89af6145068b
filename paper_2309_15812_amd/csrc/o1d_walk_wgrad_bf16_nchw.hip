// Walk kernels: weight gradient, bf16 storage, nchw.
#include "o1d_walk_kernels.h"

namespace o1d {

hipError_t launch_walk_wgrad_bf16_nchw(const walk::Plan& pl, const void* x, const void* dy, const float* theta,
                                      float* partial, hipStream_t stream) {
  return walk::wgrad_t<uint16_t, walk::kNCHW>(pl, x, dy, theta, partial, stream);
}

}  // namespace o1d
