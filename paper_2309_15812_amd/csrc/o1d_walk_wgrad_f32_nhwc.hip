// Walk kernels: weight gradient, f32 storage, nhwc.
#include "o1d_walk_kernels.h"

namespace o1d {

hipError_t launch_walk_wgrad_f32_nhwc(const walk::Plan& pl, const void* x, const void* dy, const float* theta,
                                      float* partial, hipStream_t stream) {
  return walk::wgrad_t<float, walk::kNHWC>(pl, x, dy, theta, partial, stream);
}

}  // namespace o1d
