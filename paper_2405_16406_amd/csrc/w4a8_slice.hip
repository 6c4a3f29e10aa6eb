// K-sliced tile kernels (gemm_slice.h): 8-bit activation codes.
#include "gemm_slice.h"

namespace sq {

hipError_t launch_w4a8_slice(const GemmArgs& g, const SlicePlan& p, hipStream_t stream) {
  return launch_slice_plan<kW4A8>(g, p, stream);
}

}  // namespace sq
