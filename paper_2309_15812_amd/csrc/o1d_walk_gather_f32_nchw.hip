// Walk kernels: forward pass and input gradient, f32 storage, nchw.
#include "o1d_walk_kernels.h"

namespace o1d {

hipError_t launch_walk_gather_f32_nchw(const walk::Plan& pl, const void* in, const void* w, const float* theta,
                                       void* out, hipStream_t stream) {
  return walk::gather_t<float, walk::kNCHW>(pl, in, w, theta, out, stream);
}

}  // namespace o1d
