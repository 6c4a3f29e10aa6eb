// Rotation + quantization of many rows of K = 172 * 64 (H_172 (x) S_64): activations
// (asymmetric 4- or 8-bit codes) and weight rows (symmetric 4-bit codes and their sum).
//
// View a row as X[i_a][i_b] (a x b, i_b contiguous): the result is H_a^T X S_b, computed as
// its transpose S_b^T X^T H_a.  Dense stage on the fp16 matrix cores
// (v_mfma_f32_32x32x16_f16: tile M = 32 i_b, N = 32 j_a, 16 i_a; the inputs are exact fp16 and
// H is +-1, so every product is exact and only the fp32 accumulation rounds), Sylvester
// stages over i_b in registers.
//
// Persistent: two waves share a row, a workgroup of 8 waves (two per SIMD) works on 4 rows at
// a time, one LDS slot per row, one workgroup per CU.
//   * slot: the row as APAD lines of 128 bytes (64 fp16, one i_a each), lines A..APAD-1
//     zero; on odd lines the two 64-byte halves are swapped, so that the 8 lines one
//     transposing read touches fall evenly on the two bank halves;
//   * A fragments (8 consecutive i_a of one column i_b) come from two ds_read_b64_tr_b16:
//     within each 16-lane group the instruction hands lane i element e = word i % 4 of the
//     8-byte segment addressed by lane 4e + i / 4, so lane s addresses line
//     kbase + 4t + s / 4, columns 4 (s % 4) .. +3 of its half (t = 0, 1: k 0-3 and 4-7);
//   * the B fragments of H_A (fp16 +-1) sit in LDS, built once per workgroup (some 5 us, which
//     is why few rows take the one-row kernel); each wave of the pair takes NT/2 of the MFMA
//     N tiles (the columns j_a), so neither wave needs the other's values;
//   * the next rows are loaded with 16-byte loads into registers while the current rows
//     are transformed, and written to their slots once both waves of a row have read it;
//   * one lane-half stage by v_permlane32_swap; per-row min/max (the two waves of a row meet
//     in LDS); codes use one fma per value and v_cvt_pk_u8_f32 (round half to even), which
//     can move a code by one only within 2^-12 of a rounding boundary (kMaxOffset);
//   * the two waves of a row synchronise with each other only (progress counters in LDS),
//     never with the other rows' waves, so each pair starts as soon as its own row is in.
// Bound by vector issue, for weight rows too.  Measured on MI355X (us): activations 1024 rows
// 12.9, 2048 rows 19.8, 4096 rows 32.8 (3.4 TB/s of rows
// and codes); weights [4096 x 11008] 37.9, against 7707 in the generic kernel.
#include "rot_device.h"
#include "sq_internal.h"

namespace sq {
namespace {

__device__ __forceinline__ void bfly(float& lo, float& hi) {
  const float u = lo, w = hi;
  lo = __fadd_rn(u, w);
  hi = __fsub_rn(u, w);
}

template <int A, int APAD, int NT>
struct Pair {
  static constexpr int B = 64;
  static constexpr int K = A * B;
  static constexpr int KS = APAD / 16;        // k-steps of the dense stage over i_a
  static constexpr int MT = 2;                // M tiles (32 i_b each)
  static constexpr int NTW = NT / 2;          // N tiles per wave
  static constexpr int ROWS = 4;              // rows per workgroup iteration
  static constexpr int THREADS = 64 * 2 * ROWS;
  static constexpr int CHUNKS = K / 8;                   // 16-byte chunks of a row
  static constexpr int PF = (CHUNKS + 127) / 128;        // chunks per lane of the wave pair
  static constexpr int HFRAG = KS * NT * 64;             // 16-byte B fragments
  static constexpr int SLOT = APAD * 128;                // bytes of one staged row
  static constexpr int ZERO_CHUNKS = (APAD - A) * 8;     // zero padding lines of a slot
  static constexpr int RED = 2 * ROWS * 2 * 2;           // floats: [parity][row][wave][min,max]
  static constexpr int FLAGS = 3 * ROWS * 2;             // ints: [kind][row][wave] progress counters
  static constexpr int SUMS = 2 * ROWS * 2;              // ints: [parity][row][wave] code sums (kSym4)
  static constexpr int LDS = HFRAG * 16 + ROWS * SLOT + RED * 4 + FLAGS * 4 + SUMS * 4;
  static_assert(NT % 2 == 0 && NT * 32 >= A, "N tiles");
  static_assert(APAD % 16 == 0 && APAD >= A && A % 4 == 0 && A * A % 16 == 0, "padding, whole chunks of H");
  static_assert(ZERO_CHUNKS <= 128, "one zero chunk per thread of a wave pair");
};

// Progress counter of wave `me` of a row pair: published after the wave's LDS writes, and
// awaited (counter of the partner wave >= target) before reading what the partner wrote.
__device__ __forceinline__ void pair_publish(int* flag, int value) {
  __hip_atomic_store(flag, value, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void pair_wait(const int* flag, int target) {
  while (__hip_atomic_load(flag, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP) < target)
    __builtin_amdgcn_s_sleep(1);
}

template <int A, int APAD, int NT, bool DBG, int BITS, bool VAR>
__global__ void __launch_bounds__(512, 2)
had_quant_pair(const uint16_t* x, int64_t ldx, const int8_t* H, int64_t nrows, uint8_t* q, float* alpha_out,
               RotQuantArgs args) {
  args.x = x;
  args.ldx = ldx;
  args.H = H;
  args.rows = nrows;
  args.q = q;
  args.alpha = alpha_out;
  using C = Pair<A, APAD, NT>;
  constexpr int B = C::B;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  v8h* hf = reinterpret_cast<v8h*>(smem);
  unsigned char* slots = smem + C::HFRAG * 16;
  float* red = reinterpret_cast<float*>(smem + C::HFRAG * 16 + C::ROWS * C::SLOT);
  int* flags = reinterpret_cast<int*>(smem + C::HFRAG * 16 + C::ROWS * C::SLOT + C::RED * 4);
  int* sums = flags + C::FLAGS;
  constexpr bool SYM = BITS == kSym4;
  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int p = wave >> 1;  // row slot
  const int h = wave & 1;   // which half of the N tiles
  const int g = lane >> 5;
  const int c = lane & 31;
  const int pl = h * 64 + lane;  // lane index within the wave pair (row staging)
  const int64_t rows = args.rows;
  const int64_t nsets = (rows + C::ROWS - 1) / C::ROWS;
  int64_t rs = blockIdx.x;
  if (rs >= nsets) return;  // uniform over the workgroup

  // ---- row staging: the wave pair loads chunk pl + 128 j of its row (16 bytes each)
  unsigned char* slot = slots + p * C::SLOT;
  v4u pf[C::PF];
  auto load_row = [&](int64_t r) {
    const v4u* xr = reinterpret_cast<const v4u*>(args.x + r * args.ldx);
#pragma unroll
    for (int j = 0; j < C::PF; ++j) {
      const int i = pl + 128 * j;
      pf[j] = xr[i < C::CHUNKS ? i : C::CHUNKS - 1];
    }
  };
  auto store_row = [&]() {
    if constexpr (VAR) {
      if (args.signs) {  // S flips element signs as the row goes to its slot
#pragma unroll
        for (int j = 0; j < C::PF; ++j) {
          const int i = pl + 128 * j;
          pf[j] ^= sign_mask(args.signs + 8 * (i < C::CHUNKS ? i : C::CHUNKS - 1));
        }
      }
    }
#pragma unroll
    for (int j = 0; j < C::PF; ++j) {
      const int i = pl + 128 * j;  // line i / 8, chunk i % 8; odd lines swap their halves
      if (i < C::CHUNKS) reinterpret_cast<v4u*>(slot)[i ^ ((i & 8) >> 1)] = pf[j];
    }
  };
  // ---- H_A (int8 [A][A]) with coalesced 16-byte loads, issued before the first rows so
  //      that waiting for it does not wait for them; staged as bytes in the (still empty)
  //      slot area, from which the MFMA B fragments are built while the rows are in flight
  constexpr int HCH = A * A / 16;                         // 16-byte chunks of H
  constexpr int HPT = (HCH + C::THREADS - 1) / C::THREADS;
  static_assert(HCH * 16 <= C::ROWS * C::SLOT, "H staging fits the slots");
  v4u hv[HPT];
#pragma unroll
  for (int j = 0; j < HPT; ++j) {
    const int i = threadIdx.x + j * C::THREADS;
    if (i < HCH) {
      __builtin_memcpy(&hv[j], args.H + 16 * i, 16);  // any alignment
    }
  }
  {  // the first rows are in flight while D is built
    const int64_t r0 = rs * C::ROWS + p;
    load_row(r0 < rows ? r0 : rows - 1);
  }
#pragma unroll
  for (int j = 0; j < HPT; ++j) {
    const int i = threadIdx.x + j * C::THREADS;
    if (i < HCH) reinterpret_cast<v4u*>(slots)[i] = hv[j];
  }
  if (threadIdx.x < C::FLAGS) flags[threadIdx.x] = 0;
  __syncthreads();

  // ---- H_A as MFMA B fragments: hf[(ks*NT + nt)*64 + l][e] = H[k][n] with k = ks*16 +
  //      8*(l/32) + e and n = nt*32 + l%32; zero where k or n >= A.  A thread owns one column
  //      (nt, l) of the staged bytes.
  {
    const int8_t* hs = reinterpret_cast<const int8_t*>(slots);
    for (int i = threadIdx.x; i < NT * 64; i += C::THREADS) {
      const int l = i & 63;
      const int nt = i >> 6;
      const int ja = nt * 32 + (l & 31);
      const int g8 = 8 * (l >> 5);
      const int8_t* hcol = hs + (ja < A ? ja : A - 1);
#pragma unroll
      for (int ks = 0; ks < C::KS; ++ks) {
        v8h f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const int ia = ks * 16 + g8 + e;
          const float hv1 = static_cast<float>(hcol[(ia < A ? ia : A - 1) * A]);
          f[e] = (ia < A && ja < A) ? static_cast<_Float16>(hv1) : static_cast<_Float16>(0.0f);
        }
        hf[(ks * NT + nt) * 64 + l] = f;
      }
    }
  }
  __syncthreads();  // the staged bytes are no longer read: the slots take the rows
  if (pl < C::ZERO_CHUNKS)  // the pair's padding lines i_a >= A: zero, never rewritten
    reinterpret_cast<v4u*>(slot)[A * 8 + pl] = v4u{0u, 0u, 0u, 0u};
  // flags[k*2*ROWS + p*2 + h]: k = 0: min/max of iteration it published (it + 1);
  //                            k = 1: rows of iteration it stored to the slot (it + 1)
  //                            k = 2: code sums of iteration it published (it + 1)
  int* const mine0 = flags + p * 2 + h;
  int* const mine1 = flags + 2 * C::ROWS + p * 2 + h;
  const int* const other0 = flags + p * 2 + (h ^ 1);
  const int* const other1 = flags + 2 * C::ROWS + p * 2 + (h ^ 1);
  // each pair starts as soon as its own first row is in its slot (counter value 1 before
  // iteration 0; later iterations publish it + 1 for the rows of iteration it + 1)
  store_row();
  if (lane == 0) pair_publish(mine1, 1);
  pair_wait(other1, 1);

  // transposing reads of A fragments: lane (group G = lane/16, s = lane%16) addresses line
  // 8*(G/2) + 4t + s/4 (+ 16 ks) and columns 32*mt + 16*(G%2) + 4*(s%4), whose half is
  // swapped when the line is odd (s/4 odd)
  const int tg = lane >> 4, ts = lane & 15;
  const int tq = ts >> 2;
  uint32_t tbase[C::MT];
#pragma unroll
  for (int mt = 0; mt < C::MT; ++mt)
    tbase[mt] = static_cast<uint32_t>(p * C::SLOT + (8 * (tg >> 1) + tq) * 128 +
                                      ((32 * (mt ^ (tq & 1))) + 16 * (tg & 1) + 4 * (ts & 3)) * 2);
  auto frag = [&](int mt, int ks) {
    const unsigned char* a0 = slots + tbase[mt] + ks * 16 * 128;
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) v4s*>(reinterpret_cast<uintptr_t>(a0)));
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
        reinterpret_cast<__attribute__((address_space(3))) v4s*>(reinterpret_cast<uintptr_t>(a0 + 4 * 128)));
    return __builtin_bit_cast(v8h, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
  };

  const float s_n = args.inv_sqrt_n;
  for (int it = 0; rs < nsets; ++it, rs += gridDim.x) {
    const int64_t row = rs * C::ROWS + p;
    const bool valid = row < rows;
    const bool more = rs + gridDim.x < nsets;
    if (more) {  // next rows: in flight during this iteration
      const int64_t nr = (rs + gridDim.x) * C::ROWS + p;
      load_row(nr < rows ? nr : rows - 1);
    }

    // ---- dense stage: acc[mt][nt] = X2^T H for i_b tile mt, H column tile h*NTW + nt;
    //      both M tiles' fragments read a k-step ahead
    v16f acc[C::MT][C::NTW];
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < C::NTW; ++nt)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[mt][nt][r] = 0.0f;
    {
      // A and B fragments of k-step ks + 1 are read while the MFMAs of k-step ks run
      v8h a0[C::MT], a1[C::MT], b0[C::NTW], b1[C::NTW];
      const v8h* hb = hf + h * C::NTW * 64 + lane;
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt) a0[mt] = frag(mt, 0);
#pragma unroll
      for (int nt = 0; nt < C::NTW; ++nt) b0[nt] = hb[nt * 64];
      static_for<C::KS>([&](auto kc) {
        constexpr int ks = decltype(kc)::value;
        v8h(&cur)[C::MT] = (ks & 1) ? a1 : a0;
        v8h(&nxt)[C::MT] = (ks & 1) ? a0 : a1;
        v8h(&bcur)[C::NTW] = (ks & 1) ? b1 : b0;
        v8h(&bnxt)[C::NTW] = (ks & 1) ? b0 : b1;
        if constexpr (ks + 1 < C::KS) {
#pragma unroll
          for (int mt = 0; mt < C::MT; ++mt) nxt[mt] = frag(mt, ks + 1);
#pragma unroll
          for (int nt = 0; nt < C::NTW; ++nt) bnxt[nt] = hb[((ks + 1) * NT + nt) * 64];
        }
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < C::NTW; ++nt)
            acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_f16(cur[mt], bcur[nt], acc[mt][nt], 0, 0, 0);
      });
    }

    // ---- Sylvester stages over i_b: register bits 0, 1, 3, 4; M tile bit 5; lane half bit 2
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < C::NTW; ++nt)
#pragma unroll
        for (int rb = 1; rb < 16; rb <<= 1)
#pragma unroll
          for (int r = 0; r < 16; ++r)
            if ((r & rb) == 0) {
              float lo = acc[mt][nt][r], hi = acc[mt][nt][r + rb];
              bfly(lo, hi);
              acc[mt][nt][r] = lo;
              acc[mt][nt][r + rb] = hi;
            }
#pragma unroll
    for (int nt = 0; nt < C::NTW; ++nt)
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        float lo = acc[0][nt][r], hi = acc[1][nt][r];
        bfly(lo, hi);
        acc[0][nt][r] = lo;
        acc[1][nt][r] = hi;
      }
    // lane-half stage (i_b bit 2): v_permlane32_swap of registers r and r + 8 (r < 8) puts
    // both bit-2 partners of register r (lanes 0-31) or r + 8 (lanes 32-63) in one lane;
    // the butterfly then leaves lane (c, g) holding i_b = mt*32 + 16g + j in acc[mt][nt][j],
    // j = 8q + 4*bit2 + e, sixteen consecutive positions
#pragma unroll
    for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
      for (int nt = 0; nt < C::NTW; ++nt) {
        float o[16];
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(acc[mt][nt][r]),
                                                           __float_as_uint(acc[mt][nt][r + 8]), false, false);
          const float x0 = __uint_as_float(sw[0]);  // bit 2 clear
          const float x1 = __uint_as_float(sw[1]);  // bit 2 set
          const int j = 8 * (r >> 2) + (r & 3);
          o[j] = __fadd_rn(x0, x1);
          o[j + 4] = __fsub_rn(x0, x1);
        }
#pragma unroll
        for (int j = 0; j < 16; ++j) acc[mt][nt][j] = o[j];
      }

    // ---- per-row min/max over real columns (a lane's columns past A hold zeros: merged
    //      per tile under one condition); the two waves of the row meet in LDS
    float mn = INFINITY, mx = -INFINITY;
#pragma unroll
    for (int nt = 0; nt < C::NTW; ++nt) {
      float tmn = SYM ? 0.0f : acc[0][nt][0], tmx = SYM ? 0.0f : acc[0][nt][0];
#pragma unroll
      for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          if constexpr (SYM) {
            tmx = fmaxf(tmx, fabsf(acc[mt][nt][r]));
          } else {
            tmn = fminf(tmn, acc[mt][nt][r]);
            tmx = fmaxf(tmx, acc[mt][nt][r]);
          }
        }
      if ((h * C::NTW + nt) * 32 + 32 <= A || (h * C::NTW + nt) * 32 + c < A) {
        mn = fminf(mn, tmn);
        mx = fmaxf(mx, tmx);
      }
    }
    mn = wave_min(mn);
    mx = wave_max(mx);
    // the two waves of the row meet: parity buffers, so a wave can be one iteration ahead
    float* rd = red + (it & 1) * (C::ROWS * 4);
    if (lane == 0) {
      rd[(p * 2 + h) * 2] = mn;
      rd[(p * 2 + h) * 2 + 1] = mx;
      pair_publish(mine0, it + 1);
    }
    pair_wait(other0, it + 1);  // also: the partner is done reading the slot
    mn = fminf(rd[p * 4], rd[p * 4 + 2]);
    mx = fmaxf(rd[p * 4 + 1], rd[p * 4 + 3]);
    if (more) {
      store_row();
      if (lane == 0) pair_publish(mine1, it + 2);
    }
    if constexpr (SYM) {
      const float alpha = sym_alpha(__fmul_rn(mx, s_n));
      const float inv = __fdiv_rn(1.0f, alpha);
      uint8_t* qrow = args.q + row * (C::K / 2);
      uint32_t sum8 = 0;
      int count = 0;
#pragma unroll
      for (int nt = 0; nt < C::NTW; ++nt) {
        const int ja = (h * C::NTW + nt) * 32 + c;
        uint32_t ts8 = 0;
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
          const uint32_t w0 = code_word<VAR, BITS>(acc[mt][nt], 0, s_n, inv, ts8);
          const uint32_t w1 = code_word<VAR, BITS>(acc[mt][nt], 8, s_n, inv, ts8);
          if (valid && ja < A) *reinterpret_cast<uint2*>(qrow + (ja * B + mt * 32 + 16 * g) / 2) = make_uint2(w0, w1);
        }
        sum8 += ja < A ? ts8 : 0u;
        count += ja < A ? 16 * C::MT : 0;
      }
      // the two waves' code sums meet in LDS (parity buffers, as for the min/max)
      const int sum = wave_sum(static_cast<int>(sum8) - 8 * count);
      int* const sm = sums + (it & 1) * (C::ROWS * 2) + p * 2;
      if (lane == 0) {
        sm[h] = sum;
        pair_publish(flags + 4 * C::ROWS + p * 2 + h, it + 1);
      }
      if (h == 0) {
        pair_wait(flags + 4 * C::ROWS + p * 2 + 1, it + 1);
        if (valid && lane == 0) {
          args.alpha[row] = alpha;
          args.rowsum[row] = sum + sm[1];
        }
      }
    } else {
      if constexpr (VAR) {  // clipped range [r min, r max]
        mn = __fmul_rn(mn, args.clip);
        mx = __fmul_rn(mx, args.clip);
      }

      // eq. 1 in the unscaled domain; reported alpha, beta carry the 1/sqrt(K) scale
      const float r_u = __fsub_rn(mx, mn);
      const float a_u = __fdiv_rn(r_u, BITS == 8 ? 255.0f : 15.0f);
      const bool cst = __fmul_rn(a_u, s_n) < kMinNormal;
      const float inv_u = cst ? 0.0f : __fdiv_rn(1.0f, a_u);
      float nb = -__fmul_rn(mn, inv_u);
      if (valid && h == 0 && lane == 0) {
        args.alpha[row] = cst ? 1.0f : __fmul_rn(a_u, s_n);
        args.beta[row] = __fmul_rn(mn, s_n);
      }
      if constexpr (DBG) {
#pragma unroll
        for (int nt = 0; nt < C::NTW; ++nt) {
          const int ja = (h * C::NTW + nt) * 32 + c;
          if (valid && ja < A) {
#pragma unroll
            for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
              for (int j = 0; j < 16; ++j)
                args.dbg[row * C::K + ja * B + mt * 32 + 16 * g + j] = __fmul_rn(acc[mt][nt][j], s_n);
          }
        }
      }
      if (fabsf(nb) > kMaxOffset) {  // the same for the whole row
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt)
#pragma unroll
          for (int nt = 0; nt < C::NTW; ++nt)
#pragma unroll
            for (int j = 0; j < 16; ++j) acc[mt][nt][j] = __fsub_rn(acc[mt][nt][j], mn);
        nb = 0.0f;
      }

      // ---- codes: lane (c, g) holds i_b = mt*32 + 16g + j (j = 0..15) of column j_a: bytes
      // via v_cvt_pk_u8_f32 (even j in ev, odd j in od), ev | od << 4 is then four
      // nibble-packed bytes; 8-byte store at output position j_a*64 + mt*32 + 16g.
      uint8_t* qrow = args.q + row * (C::K * BITS / 8);
#pragma unroll
      for (int nt = 0; nt < C::NTW; ++nt) {
        const int ja = (h * C::NTW + nt) * 32 + c;
#pragma unroll
        for (int mt = 0; mt < C::MT; ++mt) {
          const int pos = ja * B + mt * 32 + 16 * g;
          if constexpr (BITS == 8) {  // one code per byte: 16-byte store
            uint32_t w[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int j = 0; j < 16; ++j) w[j >> 2] = __builtin_amdgcn_cvt_pk_u8_f32(code_arg<VAR, BITS>(__fmaf_rn(acc[mt][nt][j], inv_u, nb)), j & 3, w[j >> 2]);
            if (valid && ja < A) *reinterpret_cast<uint4*>(qrow + pos) = make_uint4(w[0], w[1], w[2], w[3]);
          } else {
            uint32_t none = 0;
            const uint32_t w0 = code_word<VAR, BITS>(acc[mt][nt], 0, inv_u, nb, none);
            const uint32_t w1 = code_word<VAR, BITS>(acc[mt][nt], 8, inv_u, nb, none);
            if (valid && ja < A) *reinterpret_cast<uint2*>(qrow + pos / 2) = make_uint2(w0, w1);
          }
        }
      }
    }
    if (more) pair_wait(other1, it + 2);  // the slot holds the next row, both halves
  }
}

template <bool DBG, int BITS, bool VAR>
hipError_t launch_pair(const RotQuantArgs& a, hipStream_t stream) {
  using C = Pair<172, 176, 6>;
  constexpr auto kern = had_quant_pair<172, 176, 6, DBG, BITS, VAR>;
  const hipError_t init = set_max_lds<kern>(C::LDS);
  if (init != hipSuccess) return init;
  const int64_t sets = (a.rows + C::ROWS - 1) / C::ROWS;
  int n = 0;
  const int64_t cap = device_cus(&n) == hipSuccess ? n : 256;  // a wrong count costs rounds only
  const unsigned grid = static_cast<unsigned>(sets < cap ? sets : cap);
  return launch(kern, dim3(grid), dim3(C::THREADS), C::LDS, stream, a.x, a.ldx, a.H, a.rows, a.q, a.alpha, a);
}

template <int BITS, bool VAR>
hipError_t launch_pair_dbg(const RotQuantArgs& a, hipStream_t stream) {
  return a.dbg ? launch_pair<true, BITS, VAR>(a, stream) : launch_pair<false, BITS, VAR>(a, stream);
}

}  // namespace

hipError_t launch_had_quant_pair(const RotQuantArgs& a, hipStream_t stream) {
  const bool var = a.clip != 1.0f || a.signs != nullptr;
  if (a.bits == 8) return var ? launch_pair_dbg<8, true>(a, stream) : launch_pair_dbg<8, false>(a, stream);
  return var ? launch_pair_dbg<4, true>(a, stream) : launch_pair_dbg<4, false>(a, stream);
}

hipError_t launch_pack_pair(const RotQuantArgs& a, hipStream_t stream) {
  return a.signs ? launch_pair<false, kSym4, true>(a, stream) : launch_pair<false, kSym4, false>(a, stream);
}

}  // namespace sq
