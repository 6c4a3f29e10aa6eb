// Device helpers shared by the rotation + quantization kernels: code forms and sign masks.
#pragma once

#include "gemm_device.h"
#include "sq_device.h"

namespace sq {

typedef _Float16 v8h __attribute__((ext_vector_type(8)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef short v4s __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));

// Code width of a kernel: 4 or 8 (asymmetric activation codes), or kSym4: the symmetric
// 4-bit codes of weight rows (sq_pack_w4), quantized from the scaled values in the generic
// kernel's steps, v = y / sqrt(K), t = v (1 / alpha), code = clamp(rint(t), -7, 7).
constexpr int kSym4 = -4;

// code + 8 (1 .. 15, exact) of one unscaled value; a NaN takes the lowest code
__device__ __forceinline__ float sym_code8(float y, float s_n, float inv) {
  const float t = __fmul_rn(__fmul_rn(y, s_n), inv);
  return __fadd_rn(__builtin_rintf(__builtin_amdgcn_fmed3f(t, -7.0f, 7.0f)), 8.0f);
}

// VAR: a clipped range needs the code argument clamped to [0, L] (v_cvt_pk_u8_f32 alone
// saturates at 255 only)
template <bool VAR, int BITS>
__device__ __forceinline__ float code_arg(float t) {
  if constexpr (VAR) return __builtin_amdgcn_fmed3f(t, 0.0f, BITS == 8 ? 255.0f : 15.0f);
  return t;
}

// Codes are one fma, t = v (1 / alpha) + off with off = -fl(min / alpha): the rounding of off
// shifts a row's arguments by up to |off| 2^-24 of a step.  Rows whose range is so small against
// their values that |off| exceeds this bound subtract the minimum first (eq. 1's own steps, off
// becomes 0); with the others no argument moves by more than 2^-12 of a step, so it stays below
// 15.5 and 4-bit codes need no clamp, whatever the row.
constexpr float kMaxOffset = 4096.0f;

// Eight values' 4-bit codes, even positions in the low nibbles; kSym4: two's complement, and
// the sum of (code + 8) added to sum8
template <bool VAR, int BITS>
__device__ __forceinline__ uint32_t code_word(const v16f& y, int j0, float scale, float off, uint32_t& sum8) {
  uint32_t ev = 0, od = 0;
#pragma unroll
  for (int s = 0; s < 4; ++s) {
    const float a = y[j0 + 2 * s], b = y[j0 + 2 * s + 1];
    if constexpr (BITS == kSym4) {  // scale: 1 / sqrt(K), off: 1 / alpha
      ev = __builtin_amdgcn_cvt_pk_u8_f32(sym_code8(a, scale, off), s, ev);
      od = __builtin_amdgcn_cvt_pk_u8_f32(sym_code8(b, scale, off), s, od);
    } else {  // scale: 1 / alpha, off: -min / alpha
      ev = __builtin_amdgcn_cvt_pk_u8_f32(code_arg<VAR, BITS>(__fmaf_rn(a, scale, off)), s, ev);
      od = __builtin_amdgcn_cvt_pk_u8_f32(code_arg<VAR, BITS>(__fmaf_rn(b, scale, off)), s, od);
    }
  }
  if constexpr (BITS == kSym4) {
    sum8 = __builtin_amdgcn_sad_u8(ev, 0u, sum8);
    sum8 = __builtin_amdgcn_sad_u8(od, 0u, sum8);
    return (ev | (od << 4)) ^ 0x88888888u;  // c + 8 -> c
  }
  return ev | (od << 4);
}

// The sign flips of S (random Hadamard S H, Sec. 2.2) of a 16-byte chunk as an fp16 sign-bit
// mask, from the chunk's 8 int8 entries of S (+-1: bit 7 of byte e is the sign of element e;
// any alignment)
__device__ __forceinline__ v4u sign_mask(const int8_t* p) {
  uint2 s;
  __builtin_memcpy(&s, p, 8);
  return v4u{((s.x << 8) & 0x8000u) | ((s.x << 16) & 0x80000000u), ((s.x >> 8) & 0x8000u) | (s.x & 0x80000000u),
             ((s.y << 8) & 0x8000u) | ((s.y << 16) & 0x80000000u), ((s.y >> 8) & 0x8000u) | (s.y & 0x80000000u)};
}

}  // namespace sq
