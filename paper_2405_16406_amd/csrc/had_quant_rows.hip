// Rotation + per-row quantization of rows of length K = a * b with a registered dense order:
// R4 on activation rows (asymmetric 4- or 8-bit codes) and folded into weight rows (symmetric
// 4-bit codes with their sum).
//
// View a row as X[i_a][i_b] (a x b, i_b contiguous): the result is H_a^T X S_b.  The Sylvester
// factor splits as S_b = S_F (x) S_cols, so with the row as AD = a F lines of `cols` values the
// rotation is D (x) S_cols with D = H_a (x) S_F over the line index: a dense stage on the fp16
// matrix cores (v_mfma_f32_32x32x16_f16; the inputs are exact fp16 and D is +-1, so every
// product is exact and only the fp32 accumulation rounds) and butterflies over the columns.
//   * One workgroup per row and one row per workgroup (workgroups that share a CU cover each
//     other's loads; a loop over rows with the next one's copies under the butterflies was
//     4 - 20 % slower up to 2048 rows); one wave per 32 output lines over all columns, so
//     every butterfly stays in the wave: register bits 0, 1, 3, 4, the tiles of a wave, and
//     one lane-half stage by v_permlane32_swap, after which a lane holds 16 consecutive
//     columns of a tile.
//   * H_28 (x) S_512 and S_1024: F = 4, 112 lines in 7 k-steps.  A lane keeps the S_4 pattern
//     of its fragments and flips its sign by two H entries per k-step, which it has read as
//     bytes from global memory.  (F = 8 and 16 move one or two butterfly stages of six to eight
//     into the products at twice and four times the matrix work and LDS reads: 224 and 448
//     lines, 7 and 14 waves.)
//   * H_172 (x) S_64: F = 1, six waves of 32 output lines; H is staged in LDS as bytes, its
//     columns read back by ds_read_b64_tr_b8 (lane i of a 16-lane group gets byte i % 8 of the
//     8-byte segments that lanes 2 e + i / 8 address, e = 0 .. 7: column i of an 8 x 16 block)
//     and widened to fp16 +-1.  For more rows than kPairRounds per CU the row-pair kernel
//     (had_quant_pair.hip), which builds the fragments once, is faster.
//   * The row goes from global memory straight into LDS (buffer_load ... lds) while the
//     factor's entries are on their way.  Lines of 64 .. 256 columns; a line's 64-byte blocks
//     are permuted by its low index bits, so that the lines one transposing read touches fall
//     on distinct banks.  A fragments (8 consecutive lines of one column) come from two
//     ds_read_b64_tr_b16: within each 16-lane group that instruction hands lane i element e =
//     word i % 4 of the 8-byte segment addressed by lane 4 e + i / 4.
//   * Codes are one fma per value in the unscaled domain and v_cvt_pk_u8_f32 (rounds half to
//     even), the 1/sqrt(K) scale folded into alpha and beta; a code can differ from eq. 1's
//     steps only where its argument is within 2^-12 of a rounding boundary (kMaxOffset).
// What bounds it: a single row its own chain of load, products, butterflies, reduction and
// codes; many rows the vector issue (about 14 operations per value) and the row copies.
// Measured on MI355X, 4-bit codes (us; before: F = 8 or 16 with 7 or 14 waves and persistent
// workgroups, and the row-pair kernel at every row count):
//                          1 row   16 rows  512 rows  1024 rows  2048 rows  4096 rows
//   H_172 (x) S_64   now    4.4      4.7      7.8      (14.1)     (25.3)     (48.7)
//                    pair   9.0      9.6     10.8       12.9       19.8       32.8
//   H_28 (x) S_512   now    3.8      4.1      6.9       10.0       18.0       38.1
//                    before 4.9      5.2      9.4       14.4       23.3       44.3
//   H_28 (x) S_1024  now    6.3      6.6     12.0       20.8       44.0       82.3
//                    before 9.2      9.5     19.3       32.8       64.3      126.9
// Weight rows: [4096 x 14336] 41 (49), [8192 x 28672] 163 (290).
#include "rot_device.h"
#include "sq_internal.h"

namespace sq {
namespace {

template <int A, int F, int MT>
struct Rows {
  static constexpr int AD = A * F;               // lines of the row
  static constexpr int COLS = 32 * MT;           // fp16 per line
  static constexpr int K = AD * COLS;
  static constexpr int NT = (AD + 31) / 32;      // waves: 32 output lines each
  static constexpr int KS = (AD + 15) / 16;      // k-steps of the dense stage
  static constexpr int THREADS = 64 * NT;
  static constexpr int CPL = COLS / 8;           // 16-byte chunks per line
  static constexpr int SWZ = MT >= 4 ? 3 : MT - 1;  // 64-byte block b of line L sits at b ^ (L & SWZ)
  static constexpr int COPIES = (KS * 16 * CPL + THREADS - 1) / THREADS;  // row copies per wave
  static constexpr int SLOT = COPIES * THREADS * 16;                      // lines past AD: zeros
  static constexpr int HS = F == 1 ? NT * 32 : 0;  // bytes of a staged row of H
  static constexpr int HBYTES = KS * 16 * HS;      // rows past A are read, never written: any sign
  static constexpr int HCH = A * A / 16, HPT = (HCH + THREADS - 1) / THREADS;
  static constexpr int LDS = SLOT + HBYTES + 3 * NT * 4;  // + per-wave min, max, code sum
  static_assert(F == 4 || (F == 1 && A * A % 16 == 0 && A % 4 == 0), "two H entries per fragment, or H staged by dwords");
  static_assert((MT & (MT - 1)) == 0 && MT >= 2, "a power of two of columns");
};

// VAR: a clipping ratio and the signs S
template <int A, int F, int MT, int BITS, bool VAR>
__global__ void __launch_bounds__(64 * ((A * F + 31) / 32), 2)
had_quant_rows(const uint16_t* x, int64_t ldx, const int8_t* H, const int8_t* signs, uint8_t* q, float* alpha_out,
               float* beta_out, RotQuantArgs args) {
  args.x = x;
  args.ldx = ldx;
  args.H = H;
  args.signs = signs;
  args.q = q;
  args.alpha = alpha_out;
  args.beta = beta_out;
  constexpr bool SYM = BITS == kSym4;
  using C = Rows<A, F, MT>;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  unsigned char* const slot = smem;
  unsigned char* const hs = smem + C::SLOT;
  float* const red = reinterpret_cast<float*>(smem + C::SLOT + C::HBYTES);
  int* const sums = reinterpret_cast<int*>(red + 2 * C::NT);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = lane >> 5, c = lane & 31;
  const int n = 32 * w + c;  // output line of this lane

  // ---- H entries on their way first, then the row
  v4u hv[C::HPT];
  int8_t hb[C::KS][2];
  if constexpr (F == 1) {
#pragma unroll
    for (int j = 0; j < C::HPT; ++j) {
      const int i = threadIdx.x + j * C::THREADS;
      __builtin_memcpy(&hv[j], args.H + 16 * (i < C::HCH ? i : C::HCH - 1), 16);  // any alignment
    }
  } else {  // fragment k = 16 ks + 8 g + e lies in entries 4 ks + 2 g (e < 4) and the next
    const int na = (n < C::AD ? n : C::AD - 1) / F;
#pragma unroll
    for (int ks = 0; ks < C::KS; ++ks)
#pragma unroll
      for (int u = 0; u < 2; ++u) hb[ks][u] = args.H[(4 * ks + 2 * g + u) * A + na];
  }
  // landing chunk q of copy j: line q / CPL, block (q % CPL) / 4 in its permuted place; chunks
  // past the row land as zeros
  const int64_t row = blockIdx.x;
  auto source = [&](int j) {
    const uint32_t q = (j * C::NT + w) * 64 + lane;
    const uint32_t line = q / C::CPL, p = q % C::CPL;
    return line * C::CPL + (p ^ ((line & C::SWZ) << 2));
  };
  {
    const __amdgpu_buffer_rsrc_t rs = buf_rsrc(args.x + row * args.ldx, C::K * 2);
#pragma unroll
    for (int j = 0; j < C::COPIES; ++j) {
      auto* dst = reinterpret_cast<__attribute__((address_space(3))) void*>(
          reinterpret_cast<uintptr_t>(slot + (j * C::NT + w) * 1024));
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, static_cast<int>(source(j) * 16), 0, 0, 0);
    }
  }
  if constexpr (F == 1) {
#pragma unroll
    for (int j = 0; j < C::HPT; ++j) {
      const int i = threadIdx.x + j * C::THREADS;
      if (i < C::HCH) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {  // dword d of H: row d / (A / 4), bytes 4 (d % (A / 4)) ..
          const uint32_t d = 4 * i + t;
          *reinterpret_cast<uint32_t*>(hs + d / (A / 4) * C::HS + 4 * (d % (A / 4))) = hv[j][t];
        }
      }
    }
  }
  wait_vm_lgkm0<0>();  // the wave's own copies have landed
  asm volatile("" ::: "memory");
  if constexpr (VAR) {
    if (args.signs) {  // S flips the wave's chunks in place
#pragma unroll
      for (int j = 0; j < C::COPIES; ++j) {
        const uint32_t src = source(j);
        if (src < static_cast<uint32_t>(C::K / 8)) {
          v4u* const p = reinterpret_cast<v4u*>(slot + (j * C::NT + w) * 1024) + lane;
          *p ^= sign_mask(args.signs + 8 * src);
        }
      }
    }
  }
  __syncthreads();

  // transposing reads: lane (G = lane / 16, s = lane % 16) addresses line
  // 16 ks + 8 (G / 2) + 4 t + s / 4, columns 32 mt + 16 (G % 2) + 4 (s % 4)
  const int tg = lane >> 4, ts = lane & 15, tq = ts >> 2;
  const uint32_t tline = static_cast<uint32_t>((8 * (tg >> 1) + tq) * C::COLS * 2 + 32 * (tg & 1) + 8 * (ts & 3));
  auto frag = [&](int mt, int ks) {
    const unsigned char* a0 = slot + tline + ks * 16 * C::COLS * 2 + 64 * (mt ^ (tq & C::SWZ));
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) v4s*>(reinterpret_cast<uintptr_t>(a0)));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) v4s*>(reinterpret_cast<uintptr_t>(a0 + 4 * C::COLS * 2)));
    return __builtin_bit_cast(v8h, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };
  v4u pat;  // F == 4: S_4[e % 4][n % 4] as fp16 +-1
  if constexpr (F == 4) {
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      const int e0 = (2 * d) & 3, nt = n & 3;
      pat[d] = 0x3C003C00u | ((__popc(e0 & nt) & 1) ? 0x8000u : 0u) | ((__popc((e0 + 1) & nt) & 1) ? 0x80000000u : 0u);
    }
  }
  const uint32_t hbase = static_cast<uint32_t>((8 * (tg >> 1) + (ts >> 1)) * C::HS + 32 * w + 16 * (tg & 1) + 8 * (ts & 1));
  auto bfrag = [&](int ks) {
    v4u b;
    if constexpr (F == 1) {
      const v2i h = __builtin_amdgcn_ds_read_tr8_b64_v2i32(reinterpret_cast<__attribute__((address_space(3))) v2i*>(
          reinterpret_cast<uintptr_t>(hs + hbase + ks * 16 * C::HS)));
#pragma unroll
      for (int d = 0; d < 4; ++d) {  // sign bits of bytes 2 d, 2 d + 1 into fp16 +-1
        const uint32_t x = static_cast<uint32_t>(h[d >> 1]);
        b[d] = (__builtin_amdgcn_perm(x, x, (d & 1) ? 0x030C020Cu : 0x010C000Cu) & 0x80008000u) | 0x3C003C00u;
      }
    } else {
      const uint32_t m0 = static_cast<uint32_t>(static_cast<int>(hb[ks][0]) >> 31) & 0x80008000u;
      const uint32_t m1 = static_cast<uint32_t>(static_cast<int>(hb[ks][1]) >> 31) & 0x80008000u;
      b = v4u{pat[0] ^ m0, pat[1] ^ m0, pat[2] ^ m1, pat[3] ^ m1};
    }
    return __builtin_bit_cast(v8h, b);
  };

  auto bfly = [](float& lo, float& hi) {
    const float u = lo, v = hi;
    lo = __fadd_rn(u, v);
    hi = __fsub_rn(u, v);
  };
  const float s_n = args.inv_sqrt_n;
  const bool real = n < C::AD;
  // ---- dense stage, a k-step's fragments read ahead
  v16f acc[MT];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[mt][r] = 0.0f;
  {
    v8h a0[MT], a1[MT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt) a0[mt] = frag(mt, 0);
    static_for<C::KS>([&](auto kc) {
      constexpr int ks = decltype(kc)::value;
      v8h(&cur)[MT] = (ks & 1) ? a1 : a0;
      v8h(&nxt)[MT] = (ks & 1) ? a0 : a1;
      if constexpr (ks + 1 < C::KS) {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) nxt[mt] = frag(mt, ks + 1);
      }
      const v8h b = bfrag(ks);
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cur[mt], b, acc[mt], 0, 0, 0);
    });
  }

  // ---- Sylvester stages over the columns: register bits 0, 1, 3, 4; tile bits 5 ..; lane half bit 2
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int rb = 1; rb < 16; rb <<= 1)
#pragma unroll
      for (int r = 0; r < 16; ++r)
        if ((r & rb) == 0) {
          float lo = acc[mt][r], hi = acc[mt][r + rb];
          bfly(lo, hi);
          acc[mt][r] = lo;
          acc[mt][r + rb] = hi;
        }
#pragma unroll
  for (int mb = 1; mb < MT; mb <<= 1)
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if ((mt & mb) == 0) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          float lo = acc[mt][r], hi = acc[mt + mb][r];
          bfly(lo, hi);
          acc[mt][r] = lo;
          acc[mt + mb][r] = hi;
        }
      }
  // after the swap and butterfly lane (c, g) holds column 32 mt + 16 g + j in acc[mt][j]
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    float o[16];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
      const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[mt][r]), __float_as_uint(acc[mt][r + 8]), false, false);
      const float x0 = __uint_as_float(sw[0]), x1 = __uint_as_float(sw[1]);
      const int j = 8 * (r >> 2) + (r & 3);
      o[j] = __fadd_rn(x0, x1);
      o[j + 4] = __fsub_rn(x0, x1);
    }
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[mt][j] = o[j];
  }

  // ---- row min/max (SYM: largest magnitude) over real lines
  float mn = SYM ? 0.0f : acc[0][0], mx = SYM ? 0.0f : acc[0][0];
#pragma unroll
  for (int mt = 0; mt < MT; ++mt)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      if constexpr (SYM) {
        mx = fmaxf(mx, fabsf(acc[mt][r]));
      } else {
        mn = fminf(mn, acc[mt][r]);
        mx = fmaxf(mx, acc[mt][r]);
      }
    }
  if constexpr (!SYM) mn = wave_min(real ? mn : INFINITY);
  mx = wave_max(real ? mx : (SYM ? 0.0f : -INFINITY));
  if (lane == 0) {
    red[w] = mn;
    red[C::NT + w] = mx;
  }
  __syncthreads();
  mn = red[0];
  mx = red[C::NT];
#pragma unroll
  for (int v = 1; v < C::NT; ++v) {
    mn = fminf(mn, red[v]);
    mx = fmaxf(mx, red[C::NT + v]);
  }

  if constexpr (!SYM) {
    if (args.dbg && real) {
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 16; ++j)
          args.dbg[row * C::K + n * C::COLS + mt * 32 + 16 * g + j] = __fmul_rn(acc[mt][j], s_n);
    }
  }
  // ---- eq. 1; asymmetric: in the unscaled domain, the reported alpha and beta carry the
  // 1/sqrt(K) scale
  float alpha, beta = 0.0f, scale, off;
  if constexpr (SYM) {
    alpha = sym_alpha(__fmul_rn(mx, s_n));
    scale = s_n;
    off = __fdiv_rn(1.0f, alpha);
  } else {
    if constexpr (VAR) {  // clipped range [r min, r max]
      mn = __fmul_rn(mn, args.clip);
      mx = __fmul_rn(mx, args.clip);
    }
    const float a_u = __fdiv_rn(__fsub_rn(mx, mn), BITS == 8 ? 255.0f : 15.0f);
    const bool cst = __fmul_rn(a_u, s_n) < kMinNormal;
    scale = cst ? 0.0f : __fdiv_rn(1.0f, a_u);
    off = -__fmul_rn(mn, scale);
    alpha = cst ? 1.0f : __fmul_rn(a_u, s_n);
    beta = __fmul_rn(mn, s_n);
    if (fabsf(off) > kMaxOffset) {  // the same for the whole row
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[mt][j] = __fsub_rn(acc[mt][j], mn);
      off = 0.0f;
    }
  }
  // codes of line n, columns 32 mt + 16 g ..
  uint8_t* const qrow = args.q + row * (BITS == 8 ? C::K : C::K / 2);
  uint32_t sum8 = 0;
#pragma unroll
  for (int mt = 0; mt < MT; ++mt) {
    const int pos = n * C::COLS + mt * 32 + 16 * g;
    if constexpr (BITS == 8) {
      uint32_t wd[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int j = 0; j < 16; ++j)
        wd[j >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(code_arg<VAR, 8>(__fmaf_rn(acc[mt][j], scale, off)), j & 3, wd[j >> 2]);
      if (real) *reinterpret_cast<uint4*>(qrow + pos) = make_uint4(wd[0], wd[1], wd[2], wd[3]);
    } else {
      const uint32_t w0 = code_word<VAR, BITS>(acc[mt], 0, scale, off, sum8);
      const uint32_t w1 = code_word<VAR, BITS>(acc[mt], 8, scale, off, sum8);
      if (real) *reinterpret_cast<uint2*>(qrow + pos / 2) = make_uint2(w0, w1);
    }
  }
  if constexpr (!SYM) {
    if (threadIdx.x == 0) {
      args.alpha[row] = alpha;
      args.beta[row] = beta;
    }
  } else {
    const int sum = wave_sum(real ? static_cast<int>(sum8) - 8 * 16 * MT : 0);
    if (lane == 0) sums[w] = sum;
    __syncthreads();
    if (threadIdx.x == 0) {
      int total = sums[0];
#pragma unroll
      for (int v = 1; v < C::NT; ++v) total += sums[v];
      args.alpha[row] = alpha;
      args.rowsum[row] = total;
    }
  }
}

template <int A, int F, int MT, int BITS, bool VAR>
hipError_t launch_rows(const RotQuantArgs& a, hipStream_t stream) {
  using C = Rows<A, F, MT>;
  constexpr auto kern = had_quant_rows<A, F, MT, BITS, VAR>;
  const hipError_t init = set_max_lds<kern>(C::LDS);
  if (init != hipSuccess) return init;
  return launch(kern, dim3(static_cast<unsigned>(a.rows)), dim3(C::THREADS), C::LDS, stream, a.x, a.ldx, a.H, a.signs, a.q, a.alpha,
                a.beta, a);
}

template <int A, int F, int MT>
hipError_t launch_act(const RotQuantArgs& a, hipStream_t stream) {
  const bool var = a.clip != 1.0f || a.signs != nullptr;
  if (a.bits == 8) return var ? launch_rows<A, F, MT, 8, true>(a, stream) : launch_rows<A, F, MT, 8, false>(a, stream);
  return var ? launch_rows<A, F, MT, 4, true>(a, stream) : launch_rows<A, F, MT, 4, false>(a, stream);
}
template <int A, int F, int MT>
hipError_t launch_pack(const RotQuantArgs& a, hipStream_t stream) {
  return a.signs ? launch_rows<A, F, MT, kSym4, true>(a, stream) : launch_rows<A, F, MT, kSym4, false>(a, stream);
}

// H_172 rows per CU up to which the one-row kernel is used.  Activations, us on 256 CUs, one-row
// against row-pair: 512 rows 7.8 / 10.5, 768 rows 11.1 / 11.8, 900 rows 13.6 / 12.2, 1024 rows
// 14.1 / 12.9 (four rows per CU: one round of the pair kernel); weight rows: 512 8.9 / 12.3,
// 768 12.5 / 13.5, 1024 15.9 / 14.6, 4096 53.8 / 37.9.  (In its second round the pair kernel
// is 5 % behind again, 1100 rows 16.4 / 17.1, and ahead from 1400.)
constexpr int64_t kPairRounds = 3;
bool pair_rows(const RotQuantArgs& a) {
  int n = 0;
  return a.rows > kPairRounds * (device_cus(&n) == hipSuccess ? n : 256);
}

}  // namespace

// Rows are copied in 16-byte chunks: x is 16-byte aligned and ldx % 8 == 0 (checked by the
// entry points); the factor and the signs may have any alignment.
hipError_t launch_had_quant_rows(const RotQuantArgs& a, hipStream_t stream) {
  if ((a.bits != 4 && a.bits != 8) || a.group != a.K || a.K != static_cast<int64_t>(a.a) * a.b || a.H == nullptr)
    return hipErrorNotSupported;
  if (a.a == 172 && a.b == 64) {
    if (pair_rows(a)) return launch_had_quant_pair(a, stream);
    return launch_act<172, 1, 2>(a, stream);
  }
  if (a.a == 28 && a.b == 512) return launch_act<28, 4, 4>(a, stream);
  if (a.a == 28 && a.b == 1024) return launch_act<28, 4, 8>(a, stream);
  return hipErrorNotSupported;
}

hipError_t launch_pack_rows(const RotQuantArgs& a, hipStream_t stream) {
  if (a.K != static_cast<int64_t>(a.a) * a.b || a.H == nullptr) return hipErrorNotSupported;
  if (a.a == 172 && a.b == 64) {
    if (pair_rows(a)) return launch_pack_pair(a, stream);
    return launch_pack<172, 1, 2>(a, stream);
  }
  if (a.a == 28 && a.b == 512) return launch_pack<28, 4, 4>(a, stream);
  if (a.a == 28 && a.b == 1024) return launch_pack<28, 4, 8>(a, stream);
  return hipErrorNotSupported;
}

}  // namespace sq
