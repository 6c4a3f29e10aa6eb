// K-sliced tile kernels (gemm_slice.h): 4-bit activation codes, gate/up with SiLU.
#include "gemm_slice.h"

namespace sq {

hipError_t launch_w4a4_slice_swiglu(const GemmArgs& g, const SlicePlan& p, hipStream_t stream) {
  return launch_slice_plan<kW4A4Swiglu>(g, p, stream);
}

}  // namespace sq
