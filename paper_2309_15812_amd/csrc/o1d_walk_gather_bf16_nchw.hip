// Walk kernels: forward pass and input gradient, bf16 storage, nchw.
#include "o1d_walk_kernels.h"

namespace o1d {

hipError_t launch_walk_gather_bf16_nchw(const walk::Plan& pl, const void* in, const void* w, const float* theta,
                                       void* out, hipStream_t stream) {
  return walk::gather_t<uint16_t, walk::kNCHW>(pl, in, w, theta, out, stream);
}

}  // namespace o1d
