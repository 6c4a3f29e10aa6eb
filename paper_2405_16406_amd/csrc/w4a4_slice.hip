// K-sliced tile kernels (gemm_slice.h): 4-bit activation codes.
#include "gemm_slice.h"

namespace sq {

hipError_t launch_w4a4_slice(const GemmArgs& g, const SlicePlan& p, hipStream_t stream) {
  return launch_slice_plan<kW4A4>(g, p, stream);
}

}  // namespace sq
