// Device helpers shared by the HIP kernels: the eq. 1 quantizer's exact fp32 op
// sequence, wave/workgroup reductions, fp16 conversions.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

namespace sq {

constexpr int kWave = 64;

__device__ __forceinline__ float h2f(uint16_t bits) {
  return __half2float(__ushort_as_half(bits));
}
__device__ __forceinline__ uint16_t f2h(float v) {
  return __half_as_ushort(__float2half_rn(v));
}
// fp16 bits of v rounded to nearest even, saturating at +-65504 (the largest finite fp16)
__device__ __forceinline__ uint16_t f2h_sat(float v) {
  return f2h(fminf(fmaxf(v, -65504.0f), 65504.0f));
}

// Smallest normal fp32 (2^-126).  A group whose alpha would fall below it (zero or
// subnormal: a constant group, or a range under L * 2^-126) is quantized as constant with
// alpha = 1, so 1 / alpha stays finite and every code is 0.
constexpr float kMinNormal = 1.17549435e-38f;

// Asymmetric eq. 1 parameters from a group's min and max, L = 2^bits - 1 levels (15 or 255).
//   r = mx - mn;  alpha = r / L (1 if below kMinNormal);  inv = 1 / alpha  -- each one IEEE rounding.
struct AsymParams {
  float mn, alpha, inv, levels;
};
__device__ __forceinline__ AsymParams asym_params(float mn, float mx, float levels = 15.0f) {
  const float r = __fsub_rn(mx, mn);
  const float a = __fdiv_rn(r, levels);
  const float alpha = (a < kMinNormal) ? 1.0f : a;  // zero or subnormal: constant group
  return {mn, alpha, __fdiv_rn(1.0f, alpha), levels};
}
// t = (v - mn) * inv clamped to [0, L]: rint(t) is then the code
__device__ __forceinline__ float asym_t(float v, const AsymParams& p) {
  return __builtin_amdgcn_fmed3f(__fmul_rn(__fsub_rn(v, p.mn), p.inv), 0.0f, p.levels);
}
// code = clamp(rint((v - mn) * inv), 0, L)
__device__ __forceinline__ uint32_t asym_code(float v, const AsymParams& p) {
  const float t = __fmul_rn(__fsub_rn(v, p.mn), p.inv);
  return static_cast<uint32_t>(fminf(fmaxf(rintf(t), 0.0f), p.levels));
}

// Symmetric eq. 1 (beta = 0, L = 7): alpha = amax / 7 (1 if below kMinNormal); code in [-7, 7].
__device__ __forceinline__ float sym_alpha(float amax) {
  const float a = __fdiv_rn(amax, 7.0f);
  return (a < kMinNormal) ? 1.0f : a;
}
__device__ __forceinline__ int sym_code(float v, float inv) {
  return static_cast<int>(fminf(fmaxf(rintf(__fmul_rn(v, inv)), -7.0f), 7.0f));
}

// All-reduce over the 64 lanes without LDS: quads, eights and rows of 16 by DPP, then the rows
// of a half and the halves by permlane swaps (a swap of v with itself leaves the two partners'
// values in its two results, in every lane).  The six dependent ds_bpermute of a shuffle
// reduction cost a few hundred cycles more, which kernels of one or two rows per workgroup do
// not hide.  On MI355X (us): unrotated quantization of 1 x 4096 2.20 vs 2.66, 16 x 8192 2.90 vs
// 3.23, 4096 x 4096 8.88 vs 9.25.
template <typename Op>
__device__ __forceinline__ uint32_t wave_all(uint32_t v, Op op) {
  const auto dpp = [](uint32_t u, auto ctrl) {
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(u), decltype(ctrl)::value, 0xF, 0xF, false));
  };
  v = op(v, dpp(v, std::integral_constant<int, 0xB1>{}));   // quad_perm [1,0,3,2]
  v = op(v, dpp(v, std::integral_constant<int, 0x4E>{}));   // quad_perm [2,3,0,1]
  v = op(v, dpp(v, std::integral_constant<int, 0x141>{}));  // row_half_mirror
  v = op(v, dpp(v, std::integral_constant<int, 0x140>{}));  // row_mirror
  const auto s16 = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  v = op(s16[0], s16[1]);
  const auto s32 = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return op(s32[0], s32[1]);
}
__device__ __forceinline__ float wave_min(float v) {
  return __uint_as_float(wave_all(__float_as_uint(v), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fminf(__uint_as_float(a), __uint_as_float(b)));
  }));
}
__device__ __forceinline__ float wave_max(float v) {
  return __uint_as_float(wave_all(__float_as_uint(v), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }));
}
__device__ __forceinline__ int wave_sum(int v) {
  return static_cast<int>(wave_all(static_cast<uint32_t>(v), [](uint32_t a, uint32_t b) { return a + b; }));
}

// floor(x / d) and the remainder, with magic = floor(2^32 / d) + 1 from the host (32 bits; 0 for
// d == 1).  x magic / 2^32 exceeds x / d by at most x / 2^32: its floor is at most one too many.
inline uint32_t div_magic(uint32_t d) { return d == 1 ? 0u : static_cast<uint32_t>((uint64_t{1} << 32) / d + 1); }
__device__ __forceinline__ void div_rem(uint32_t x, uint32_t d, uint32_t magic, uint32_t& quot, uint32_t& rem) {
  quot = magic ? static_cast<uint32_t>((static_cast<uint64_t>(x) * magic) >> 32) : x;
  if (quot * d > x) --quot;
  rem = x - quot * d;
}

}  // namespace sq
