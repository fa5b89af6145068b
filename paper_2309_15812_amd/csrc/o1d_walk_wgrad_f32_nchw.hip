// Walk kernels: weight gradient, f32 storage, nchw.
#include "o1d_walk_kernels.h"

namespace o1d {

hipError_t launch_walk_wgrad_f32_nchw(const walk::Plan& pl, const void* x, const void* dy, const float* theta,
                                      float* partial, hipStream_t stream) {
  return walk::wgrad_t<float, walk::kNCHW>(pl, x, dy, theta, partial, stream);
}

}  // namespace o1d
