// Device helpers shared by the GEMM translation units: vector types, buffer descriptors,
// the epilogue's rounding steps, SiLU and the operand forms of the int8 matrix products.
#pragma once

#include <cstdint>
#include <type_traits>
#include <utility>

#include "sq_device.h"

namespace sq {

typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef _Float16 v2h __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

// The epilogue rounds twice, fp32 then fp16 (round to nearest even), in both of its paths.
// fp32_result pins a value as a rounded fp32 register so that the compiler cannot fuse the
// final fma with the fp16 conversion into one single-rounding v_fma_mix.  The asm is not
// volatile: it only hides the value, and the scheduler stays free to interleave the
// independent outputs (volatile asm statements keep their program order, which serialised
// the epilogue's long-latency exp and reciprocal steps).
__device__ __forceinline__ float fp32_result(float v) {
  asm("" : "+v"(v));
  return v;
}
// two fp32 -> two fp16 (round to nearest even), packed low | high << 16
__device__ __forceinline__ uint32_t f2h2(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v2f{lo, hi}, v2h));
}

// Calls f(std::integral_constant<int, I>) for I = 0 .. N-1: indices into register arrays
// stay compile-time constants even where the unroller would give up.
template <typename F, int... Is>
__host__ __device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, Is...>) {
  (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__host__ __device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t buf_rsrc(const void* p, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, static_cast<int>(bytes), 0x00020000);
}

// SiLU(gate) * up of two dequantised fp32 outputs, as the fp16 input of down_proj:
// g u / (1 + e^-g), the quotient as a product with v_rcp_f32 (1 ulp; the result is rounded
// to fp16) instead of the IEEE division sequence, which took most of the gate/up epilogue's
// instructions; for g -> -inf the denominator is +inf, its reciprocal 0 and the product 0.
__device__ __forceinline__ float swiglu_value(float gv, float uv) {
  return __fmul_rn(__fmul_rn(gv, uv), __builtin_amdgcn_rcpf(__fadd_rn(1.0f, __expf(-gv))));
}

// 16 8-bit activation codes k0..k15 (natural order) -> signed operand in the slot order of
// the nibble expansion (k0 k2 k4 k6 | k1 k3 k5 k7 | k8 ...)
__device__ __forceinline__ v4i act8_operand(const v4u d) {
  const uint32_t f = 0x80808080u;
  return v4i{static_cast<int>(__builtin_amdgcn_perm(d[1], d[0], 0x06040200u) ^ f),
             static_cast<int>(__builtin_amdgcn_perm(d[1], d[0], 0x07050301u) ^ f),
             static_cast<int>(__builtin_amdgcn_perm(d[3], d[2], 0x06040200u) ^ f),
             static_cast<int>(__builtin_amdgcn_perm(d[3], d[2], 0x07050301u) ^ f)};
}
// s_waitcnt with vmcnt = VM (0..63: bits 3:0 and 15:14) and lgkmcnt = 0 (expcnt not waited on)
template <int VM>
__device__ __forceinline__ void wait_vm_lgkm0() {
  static_assert(VM >= 0 && VM <= 63, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt((VM & 0xF) | ((VM >> 4) << 14) | (0x7 << 4));
}

}  // namespace sq
