// int4 x int4 GEMM on the int8 matrix cores of gfx950 with the dequantising epilogue.
//
// acc[m,n] = sum_k qa[m,k] qw[n,k] (exact, int32), y = fp16(s_n (alpha_m acc + beta_m rs_n) + bias_n).
//
// Codes arrive packed two per byte (even k in the low nibble).  Both operands are
// expanded to int8 in registers just before v_mfma_i32_32x32x32_i8:
//   activations (0..15):  lo = d & 0x0F0F0F0F,         hi = (d >> 4) & 0x0F0F0F0F
//   weights (-7..7):      lo = (d << 4) & 0xF0F0F0F0,  hi = d & 0xF0F0F0F0     (= 16 * code)
// so each int8 byte holds one code (weights scaled by 16, which is exact) and the
// accumulator is 16 * acc; an arithmetic shift by 4 recovers acc exactly.  A and B are
// expanded with the same byte order, so the k permutation this introduces cancels in
// the dot product.  |16 acc| <= 16 * 15 * 7 * K < 2^31 for K < 1.2M.
//
// Prompts (w4a4_gemm_ring, this file): the packed operand tiles stream from global memory
// into an LDS ring by direct-to-LDS buffer loads, several stages ahead; each wave reads its
// fragments back with ds_read_b128, expands them with VALU and issues the MFMAs.  Tile
// shapes: 256 x 256 (8 waves of 128 x 64, or 64 x 128 with 8-bit codes), 128 x 256 (8 waves
// of 64 x 64) and, with SiLU, 256 x 128 (4 waves of 128 x 64, two workgroups per CU).
// Everything below that, and operands that 32-bit buffer offsets do not cover: the K-sliced
// tile kernel (gemm_slice.h); gemm_plan.h chooses.
#include "gemm_device.h"
#include "gemm_plan.h"
#include "sq_device.h"
#include "sq_internal.h"

namespace sq {
namespace {

// Tile order.  Consecutive workgroup ids go to different XCDs (round robin over 8), so each
// XCD is given a contiguous range of tile ids; within it the tile walks M fastest, so the
// CUs of one XCD share weight (B) tiles in their L2 and each weight tile is read from HBM
// about once.
__device__ __forceinline__ void tile_origin(int bm, int bn, int tiles_m, int total, uint32_t magic, int64_t& m0, int64_t& n0) {
  const int bid = blockIdx.x;
  const int q8 = total / 8, r8 = total % 8;
  const int xcd = bid % 8, idx = bid / 8;
  const int tile = xcd < r8 ? xcd * (q8 + 1) + idx : r8 * (q8 + 1) + (xcd - r8) * q8 + idx;
  uint32_t tn, tm;
  div_rem(tile, tiles_m, magic, tn, tm);
  m0 = static_cast<int64_t>(tm) * bm;
  n0 = static_cast<int64_t>(tn) * bn;
}

// Epilogue of the ring kernel.  Its MFMAs take the weights as the A operand, so each 32 x 32
// block is D[n][m]: lane (c, h) = (lane % 32, lane / 32) holds row m = mb + c and columns
// n = nb + 8q + 4h + e in registers r = 4q + e, i.e. four consecutive outputs of one row per
// q, written with one 8-byte store.  The accumulators hold 16 * acc (weights expanded as
// 16 * code), so alpha_m / 16 is applied:
//   y = fma(alpha_m/16, s_n * acc16, fma(beta_m, s_n rs_n, bias_n))   (bias_n = 0 without a bias).
// Per-tile row and column scales are staged in LDS during the prologue (RingScales).
template <int BM, int BN>
struct RingScales {
  // floats: rowA[BM] (alpha_m / 16), rowB[BM] (beta_m; 8-bit codes: beta_m + 128 alpha_m),
  // colS[BN] (s_n), colR[BN] (rs_n), colB[BN] (bias_n)
  static constexpr int COUNT = 2 * BM + 3 * BN;
  static constexpr int BYTES = COUNT * 4;
};

// Scale value `idx` of a tile (RingScales layout), in two steps: fetch() reads every
// candidate source at a clamped index, unconditionally, and value() selects and converts.
// The caller issues the fetches before the tile's first copies and calls value() after the
// first stage has landed: the loads are then all in flight at once and off the copies'
// path (loads in branches made the compiler wait for each before the copies went out).
// Out-of-range rows/columns give 0.
struct ScaleFetch {
  float xa, xb, wa;
  int32_t rs;
  uint16_t bias;
};
template <int BM, int BN>
__device__ __forceinline__ ScaleFetch scale_fetch(const GemmArgs& g, int idx, int64_t m0, int64_t n0) {
  const int t = idx < 2 * BM ? 0 : idx - 2 * BM;
  const int64_t m = m0 + (idx % BM), n = n0 + (t % BN);
  const int64_t mc = m < g.M ? m : g.M - 1, nc = n < g.N ? n : g.N - 1;
  // without a bias the fetch reads (and discards) the first bytes of the scales
  const uint16_t* bp = g.bias ? g.bias : reinterpret_cast<const uint16_t*>(g.wa);
  return ScaleFetch{g.xa[mc], g.xb[mc], g.wa[nc], g.rs[nc], bp[nc]};
}
template <int BM, int BN>
__device__ __forceinline__ float scale_value(const GemmArgs& g, const ScaleFetch& f, int idx, int64_t m0, int64_t n0) {
  if (idx < 2 * BM) {
    if (m0 + (idx % BM) >= g.M) return 0.0f;
    if (idx < BM) return __fmul_rn(f.xa, 0.0625f);
    return g.a8 ? __fmaf_rn(128.0f, f.xa, f.xb) : f.xb;  // 8-bit codes enter as qa - 128
  }
  const int t = idx - 2 * BM;
  if (n0 + (t % BN) >= g.N) return 0.0f;
  if (t < BN) return f.wa;
  if (t < 2 * BN) return static_cast<float>(f.rs);
  return g.bias ? h2f(f.bias) : 0.0f;
}

// Byte address in a staged output tile (rows of RB bytes, 16-byte chunks of row r XOR-ed
// with r % (RB / 16) so that the 32 rows one store instruction spans fall on different banks).
template <int RB>
__device__ __forceinline__ uint32_t stage_addr(int r, int b) {
  constexpr int CH = RB / 16;
  return static_cast<uint32_t>(r * RB + (((b >> 4) ^ (r & (CH - 1))) << 4) + (b & 15));
}

// Stores a staged BM x BNO fp16 output tile (rows m0.., columns n0o..) with whole-row 16-byte
// pieces: one store instruction covers 64 / (BNO / 8) full rows.  Rows past M are dropped by
// the buffer range.  Needs ldy % 8 == 0, a 16-byte aligned y and n0o % 8 == 0.
template <int BM, int BNO>
__device__ __forceinline__ void store_staged(const GemmArgs& g, const uint8_t* stg, int64_t m0, int64_t n0o, int wave,
                                             int waves, int lane) {
  constexpr int RB = BNO * 2, CH = RB / 16, RPI = 64 / CH;
  static_assert(CH <= 64 && 64 % CH == 0, "rows of at most 1 KB");
  const __amdgpu_buffer_rsrc_t ry = buf_rsrc(g.y, g.M * g.ldy * 2);
  const int k = lane % CH;
  for (int r0 = wave * RPI; r0 < BM; r0 += waves * RPI) {
    const int rr = r0 + lane / CH;
    const v4u v = *reinterpret_cast<const v4u*>(stg + stage_addr<RB>(rr, 16 * k));
    const int64_t m = m0 + rr;
    const uint32_t off = m < g.M ? static_cast<uint32_t>((m * g.ldy + n0o) * 2 + 16 * k) : 0x80000000u;
    __builtin_amdgcn_raw_buffer_store_b128(v, ry, static_cast<int>(off), 0, 0);
  }
}

// Checked path: edge tiles, unaligned or large outputs, and the raw accumulator output.
template <int TM, int TN, int BM, int BN>
__device__ __forceinline__ void ring_epilogue_checked(const GemmArgs& g, const v16i (&acc)[TM][TN], int64_t mw,
                                                      int64_t nw, int tm, int tn, int lane, const float* __restrict__ sc) {
  const int c = lane & 31;
  const int h = lane >> 5;
  const float* rowA = sc;
  const float* rowB = sc + BM;
  const float* colS = sc + 2 * BM;
  const float* colR = colS + BN;
  const float* colB = colR + BN;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t m = mw + i * 32 + c;
    if (m >= g.M) continue;
    const float ra = rowA[(tm + i) * 32 + c], rb = rowB[(tm + i) * 32 + c];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int cl = (tn + j) * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        const int64_t n = nw + j * 32 + 8 * (r >> 2) + 4 * h + (r & 3);
        if (n >= g.N) continue;
        const float s = colS[cl];
        const float t = __fmul_rn(s, static_cast<float>(acc[i][j][r]));
        const float yv = fp32_result(__fmaf_rn(ra, t, __fmaf_rn(rb, __fmul_rn(s, colR[cl]), colB[cl])));
        g.y[m * g.ldy + n] = f2h(yv);
        if (g.dbg_acc) g.dbg_acc[m * g.N + n] = (acc[i][j][r] >> 4) + (g.a8 ? 128 * g.rs[n] : 0);
      }
    }
  }
}

// Gate/up epilogues: wq interleaves gate and up rows in blocks of 32, so the wave's block
// pair (2p, 2p + 1) holds the gate and up outputs of the same 32 columns in the same lane
// and registers; output column = (interleaved column of the gate block) / 2 + offset.
template <int TM, int TN, int BM, int BN>
__device__ __forceinline__ void ring_epilogue_swiglu_checked(const GemmArgs& g, const v16i (&acc)[TM][TN],
                                                             int64_t mw, int64_t nw, int tm, int tn, int lane,
                                                             const float* __restrict__ sc) {
  static_assert(TN % 2 == 0, "gate/up block pairs");
  const int c = lane & 31;
  const int h = lane >> 5;
  const float* rowA = sc;
  const float* rowB = sc + BM;
  const float* colS = sc + 2 * BM;
  const float* colR = colS + BN;
  const float* colB = colR + BN;
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    const int64_t m = mw + i * 32 + c;
    if (m >= g.M) continue;
    const float ra = rowA[(tm + i) * 32 + c], rb = rowB[(tm + i) * 32 + c];
#pragma unroll
    for (int p = 0; p < TN / 2; ++p) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int off = 8 * (r >> 2) + 4 * h + (r & 3);
        const int cg = (tn + 2 * p) * 32 + off, cu = cg + 32;
        const int64_t ng = nw + 64 * p + off;  // gate column; its up column ng + 32 < N (N % 64 == 0)
        if (ng >= g.N) continue;
        const float gv = fp32_result(__fmaf_rn(ra, __fmul_rn(colS[cg], static_cast<float>(acc[i][2 * p][r])),
                                               __fmaf_rn(rb, __fmul_rn(colS[cg], colR[cg]), colB[cg])));
        const float uv = fp32_result(__fmaf_rn(ra, __fmul_rn(colS[cu], static_cast<float>(acc[i][2 * p + 1][r])),
                                               __fmaf_rn(rb, __fmul_rn(colS[cu], colR[cu]), colB[cu])));
        g.y[m * g.ldy + (nw + 64 * p) / 2 + off] = f2h(fp32_result(swiglu_value(gv, uv)));
      }
    }
  }
}

// The fast epilogue through a staged tile in LDS (stg: BM x BN fp16, or BM x BN/2 for
// gate/up, in the ring's bytes, which the caller has drained): every wave writes its block
// (same arithmetic as the other epilogues), a workgroup barrier, then the whole tile goes
// out in whole-row pieces.  Column groups q run outermost so that only one group's column
// scales are live.  Needs what store_staged needs.
template <int TM, int TN, int BM, int BN>
__device__ __forceinline__ void ring_epilogue_staged(const GemmArgs& g, const v16i (&acc)[TM][TN], int64_t m0,
                                                     int64_t n0, int tm, int tn, int lane, const float* __restrict__ sc,
                                                     uint8_t* stg, int wave, int waves) {
  const int c = lane & 31;
  const int h = lane >> 5;
  const float* rowA = sc;
  const float* rowB = sc + BM;
  const float* colS = sc + 2 * BM;
  const float* colR = colS + BN;
  const float* colB = colR + BN;
  float ra[TM], rb[TM];
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    ra[i] = rowA[(tm + i) * 32 + c];
    rb[i] = rowB[(tm + i) * 32 + c];
  }
  const bool sw = g.swiglu;
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float s[TN][4], w[TN][4], bv[TN][4];
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int cb = (tn + j) * 32 + 8 * q + 4 * h;
      const float4 sv = *reinterpret_cast<const float4*>(colS + cb);
      const float4 rv = *reinterpret_cast<const float4*>(colR + cb);
      const float4 bb = *reinterpret_cast<const float4*>(colB + cb);
      const float s4[4] = {sv.x, sv.y, sv.z, sv.w}, r4[4] = {rv.x, rv.y, rv.z, rv.w}, b4[4] = {bb.x, bb.y, bb.z, bb.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s[j][e] = s4[e];
        w[j][e] = __fmul_rn(s4[e], r4[e]);
        bv[j][e] = b4[e];
      }
    }
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      const int r0 = 4 * q;
      const int row = (tm + i) * 32 + c;
      if (sw) {
        if constexpr (TN % 2 == 0) {
#pragma unroll
          for (int p = 0; p < TN / 2; ++p) {
            uint32_t pk[2];
#pragma unroll
            for (int e2 = 0; e2 < 2; ++e2) {
              float hv[2];
#pragma unroll
              for (int u = 0; u < 2; ++u) {
                const int e = 2 * e2 + u;
                const int jg = 2 * p, ju = 2 * p + 1;
                const float tg = __fmul_rn(s[jg][e], static_cast<float>(acc[i][jg][r0 + e]));
                const float tu = __fmul_rn(s[ju][e], static_cast<float>(acc[i][ju][r0 + e]));
                const float gv = fp32_result(__fmaf_rn(ra[i], tg, __fmaf_rn(rb[i], w[jg][e], bv[jg][e])));
                const float uv = fp32_result(__fmaf_rn(ra[i], tu, __fmaf_rn(rb[i], w[ju][e], bv[ju][e])));
                hv[u] = fp32_result(swiglu_value(gv, uv));
              }
              pk[e2] = f2h2(hv[0], hv[1]);
            }
            *reinterpret_cast<v2u*>(stg + stage_addr<BN>(row, ((tn / 2 + p) * 32 + 8 * q + 4 * h) * 2)) =
                v2u{pk[0], pk[1]};
          }
        }
      } else {
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          uint32_t pk[2];
#pragma unroll
          for (int e2 = 0; e2 < 2; ++e2) {
            float yv[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
              const int e = 2 * e2 + u;
              const float t = __fmul_rn(s[j][e], static_cast<float>(acc[i][j][r0 + e]));
              yv[u] = fp32_result(__fmaf_rn(ra[i], t, __fmaf_rn(rb[i], w[j][e], bv[j][e])));
            }
            pk[e2] = f2h2(yv[0], yv[1]);
          }
          *reinterpret_cast<v2u*>(stg + stage_addr<BN * 2>(row, ((tn + j) * 32 + 8 * q + 4 * h) * 2)) =
              v2u{pk[0], pk[1]};
        }
      }
    }
  }
  __syncthreads();
  if (sw)
    store_staged<BM, BN / 2>(g, stg, m0, n0 / 2, wave, waves, lane);
  else
    store_staged<BM, BN>(g, stg, m0, n0, wave, waves, lane);
}

// ------------------------------------------------------------------ LDS-ring tile kernel
// Packed operand tiles go from global memory straight into LDS (buffer_load_dwordx4 ... lds:
// no registers, no VALU), NS stages deep, so a stage's loads are in flight for NS - 1 stages
// of MFMA work.  A stage covers 128 k (64 packed bytes per row) and is laid out as 1 KB
// blocks, one per 32 rows and pair of 16-byte chunks: lane l of the copying wave brings row
// l % 32, chunk 2p + l / 32 to byte 16 l of the block.  A wave reads a block back with one
// contiguous ds_read_b128 (no bank conflicts); each lane then holds 32 codes of one row,
// which expand into the operands of two MFMA k-steps.  Both operands use the same k-slot
// order, so the dot product is unchanged.  Rows past M or N and chunks past K are out of the
// buffer range and land as zeros.
// 8-bit activations (A8, the W4A8 setting): a stage row is 128 code bytes, 8 chunks, and the
// A blocks are one per 32 rows and (chunk pair p, half H): lane l of the copying wave brings
// row l % 32, chunk 4p + 2(l / 32) + H, so the lane (c, h) that reads it back holds exactly
// the 16 codes of k-step (p, H) that the 4-bit expansion gives it (k = 64p + 32h + 16H + e);
// v_perm_b32 puts them in the same slot order and an xor with 0x80 makes them signed.
template <int WAVES_M, int WAVES_N, int TM, int TN, int NS, bool A8 = false>
struct Ring {
  static constexpr int WAVES = WAVES_M * WAVES_N;
  static constexpr int THREADS = 64 * WAVES;
  static constexpr int BM = WAVES_M * TM * 32;
  static constexpr int BN = WAVES_N * TN * 32;
  static constexpr int ABLK = BM / (A8 ? 8 : 16);  // 1 KB blocks per stage: 32 rows x 2 (A8: 4) chunk pairs
  static constexpr int BBLK = BN / 16;
  static constexpr int ADPW = ABLK / WAVES;  // block copies per wave per stage
  static constexpr int DPW = (ABLK + BBLK) / WAVES;
  static constexpr int STAGE = (ABLK + BBLK) * 1024;
  static_assert(ADPW * WAVES == ABLK && DPW * WAVES == ABLK + BBLK, "blocks split evenly over waves");
  static_assert(NS >= 2 && (NS - 1) * DPW <= 63, "outstanding copies fit the vmcnt counter");
};

template <int TM, int TN, bool A8 = false>
struct RingPacked {  // one chunk pair (two k-steps) of the wave's A and B blocks
  v4u a[TM][A8 ? 2 : 1];
  v4u b[TN];
};

template <int TM, int TN>
struct RingOps {  // MFMA operands of one k-step
  v4i a[TM];
  v4i b[TN];
};

// Operands of k-step H (0: dwords 0-1, 1: dwords 2-3) of a packed chunk pair.
template <int H, int TM, int TN, bool A8>
__device__ __forceinline__ void expand_half(const RingPacked<TM, TN, A8>& P, RingOps<TM, TN>& E) {
#pragma unroll
  for (int i = 0; i < TM; ++i) {
    if constexpr (A8) {
      E.a[i] = act8_operand(P.a[i][H]);
    } else {
      const uint32_t d0 = P.a[i][0][2 * H], d1 = P.a[i][0][2 * H + 1];
      E.a[i] = v4i{static_cast<int>(d0 & 0x0F0F0F0Fu), static_cast<int>((d0 >> 4) & 0x0F0F0F0Fu),
                   static_cast<int>(d1 & 0x0F0F0F0Fu), static_cast<int>((d1 >> 4) & 0x0F0F0F0Fu)};
    }
  }
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const uint32_t d0 = P.b[j][2 * H], d1 = P.b[j][2 * H + 1];
    E.b[j] = v4i{static_cast<int>((d0 << 4) & 0xF0F0F0F0u), static_cast<int>(d0 & 0xF0F0F0F0u),
                 static_cast<int>((d1 << 4) & 0xF0F0F0F0u), static_cast<int>(d1 & 0xF0F0F0F0u)};
  }
}

// LDS of a ring kernel: the ring, then the tile's epilogue scales.
template <int WAVES_M, int WAVES_N, int TM, int TN, int NS, bool A8 = false>
struct RingLds {
  using R = Ring<WAVES_M, WAVES_N, TM, TN, NS, A8>;
  static constexpr int SCALES = NS * R::STAGE;  // byte offset of the scales
  static constexpr int BYTES = SCALES + RingScales<R::BM, R::BN>::BYTES;
};

template <int WAVES_M, int WAVES_N, int TM, int TN, int NS, int WPE, bool A8 = false>
__global__ void __launch_bounds__(64 * WAVES_M * WAVES_N, WPE)
w4a4_gemm_ring(const uint8_t* xq, const uint8_t* wq, int64_t M, int64_t N, int K, int tiles_m, int tiles, uint32_t magic,
               GemmArgs g) {
  g.xq = xq;
  g.wq = wq;
  g.M = M;
  g.N = N;
  g.K = K;
  using R = Ring<WAVES_M, WAVES_N, TM, TN, NS, A8>;
  using L = RingLds<WAVES_M, WAVES_N, TM, TN, NS, A8>;
  using SC = RingScales<R::BM, R::BN>;
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const scales = reinterpret_cast<float*>(lds + L::SCALES);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  uint8_t* const ring = lds;
  int64_t m0, n0;
  tile_origin(R::BM, R::BN, tiles_m, tiles, magic, m0, n0);
  const int wm = (wave / WAVES_N) * TM;  // first 32-row group of this wave in the tile
  const int wn = (wave % WAVES_N) * TN;
  const uint32_t KB = static_cast<uint32_t>(g.K / 2);
  const uint32_t KA = A8 ? 2 * KB : KB;  // activation bytes per row
  const int nstage = static_cast<int>((KB + 63) / 64);

  // Buffer ranges: offsets are 32-bit and (M + BM) * KA < 2^31 is checked on the host.
  const __amdgpu_buffer_rsrc_t rsa =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.xq), 0, static_cast<int>(g.M * KA), 0x00020000);
  const __amdgpu_buffer_rsrc_t rsb =
      __builtin_amdgcn_make_buffer_rsrc(const_cast<uint8_t*>(g.wq), 0, static_cast<int>(g.N * KB), 0x00020000);
  // Copy d of this wave is block b = wave + WAVES d of a stage: A blocks first, then B.
  uint32_t rowoff[R::DPW], colofs[R::DPW];
  static_for<R::DPW>([&](auto dc) {
    constexpr int d = decltype(dc)::value;
    const int b = wave + R::WAVES * d;
    const int bl = d < R::ADPW ? b : b - R::ABLK;
    if (A8 && d < R::ADPW) {  // block (row group, p, H): chunk 4p + 2h + H of the 128-byte row
      const int64_t row = m0 + (bl >> 2) * 32 + (lane & 31);
      rowoff[d] = static_cast<uint32_t>(row) * KA;
      colofs[d] = ((bl >> 1) & 1) * 64 + (lane >> 5) * 32 + (bl & 1) * 16;
    } else {
      const int64_t row = (d < R::ADPW ? m0 : n0) + (bl >> 1) * 32 + (lane & 31);
      rowoff[d] = static_cast<uint32_t>(row) * KB;
      colofs[d] = (bl & 1) * 32 + (lane >> 5) * 16;
    }
  });
  auto issue = [&](int st) {
    uint8_t* sb = ring + (st % NS) * R::STAGE;
    const uint32_t k0 = static_cast<uint32_t>(st) * 64;
    const bool live = st < nstage;
    static_for<R::DPW>([&](auto dc) {
      constexpr int d = decltype(dc)::value;
      constexpr bool a8blk = A8 && d < R::ADPW;
      const uint32_t col = (a8blk ? 2 * k0 : k0) + colofs[d];
      // past K, or a stage past the end (issued only to keep the copy count uniform): out of
      // range, lands as zeros
      const uint32_t off = (live && col < (a8blk ? KA : KB)) ? rowoff[d] + col : 0x80000000u;
      auto* dst = reinterpret_cast<__attribute__((address_space(3))) void*>(
          reinterpret_cast<uintptr_t>(sb + (wave + R::WAVES * d) * 1024));
      if constexpr (d < R::ADPW)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsa, dst, 16, static_cast<int>(off), 0, 0, 0);
      else
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsb, dst, 16, static_cast<int>(off), 0, 0, 0);
    });
  };
  auto read = [&](RingPacked<TM, TN, A8>& P, int st, int p) {
    const uint8_t* sb = ring + (st % NS) * R::STAGE + lane * 16;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if constexpr (A8) {
        P.a[i][0] = *reinterpret_cast<const v4u*>(sb + (wm + i) * 4096 + (2 * p) * 1024);
        P.a[i][1] = *reinterpret_cast<const v4u*>(sb + (wm + i) * 4096 + (2 * p + 1) * 1024);
      } else {
        P.a[i][0] = *reinterpret_cast<const v4u*>(sb + (wm + i) * 2048 + p * 1024);
      }
    }
#pragma unroll
    for (int j = 0; j < TN; ++j) P.b[j] = *reinterpret_cast<const v4u*>(sb + (R::ABLK + 2 * (wn + j) + p) * 1024);
  };
  // MFMAs of one k-step from E, with the next k-step's operands expanded into F in between
  constexpr int NM = TM * TN;
  constexpr int NV = (A8 ? 8 : 6) * TM + 6 * TN;
  constexpr int PER = (NV + NM - 2) / (NM - 1);
  auto mma = [&](v16i (&acc)[TM][TN], const RingOps<TM, TN>& E) {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = __builtin_amdgcn_mfma_i32_32x32x32_i8(E.b[j], E.a[i], acc[i][j], 0, 0, 0);
  };
  // ds_reads (NR of them) first, then one MFMA per PER expansion ops
  auto interleave = [&](auto nr) {
    constexpr int NR = decltype(nr)::value;
    if constexpr (NR > 0) __builtin_amdgcn_sched_group_barrier(0x100, NR, 0);
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
#pragma unroll
    for (int k = 0; k < NM - 1; ++k) {
      __builtin_amdgcn_sched_group_barrier(0x002, PER, 0);
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
    }
  };
  auto sync = [&]() {
    wait_vm_lgkm0<(NS - 2) * R::DPW>();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  v16i acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0;

  // Pipeline over k-steps (four per stage).  Packed chunk pairs are read from LDS two
  // k-steps before their first expansion, operands are expanded one k-step ahead of their
  // MFMAs, and the stage sync sits in the second k-step, after the last read of the
  // current stage's slot (which the copy issued right after it refills).
  // epilogue scales of the tile: loaded now, written to LDS after the first copies have
  // landed (the main loop's barriers publish them)
  constexpr int TT = R::THREADS;
  constexpr int SPT = (SC::COUNT + TT - 1) / TT;
  ScaleFetch sf[SPT];
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const int idx = static_cast<int>(threadIdx.x) + u * TT;
    sf[u] = scale_fetch<R::BM, R::BN>(g, idx < SC::COUNT ? idx : 0, m0, n0);
  }
  for (int s = 0; s < NS - 1; ++s) issue(s);
  sync();
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const int idx = static_cast<int>(threadIdx.x) + u * TT;
    if (idx < SC::COUNT) scales[idx] = scale_value<R::BM, R::BN>(g, sf[u], idx, m0, n0);
  }
  issue(NS - 1);
  RingPacked<TM, TN, A8> P0, P1;
  RingOps<TM, TN> E0, E1;
  read(P0, 0, 0);
  read(P1, 0, 1);
  expand_half<0>(P0, E0);

  // Branch-free steady state: the last iteration also syncs, copies (out of range) and
  // expands the stage after the end; those operands are never used.
  for (int st = 0; st < nstage; ++st) {
    constexpr std::integral_constant<int, 0> none{};
    constexpr std::integral_constant<int, (A8 ? 2 : 1) * TM + TN> all{};  // ds_reads of one read()
    mma(acc, E0);                 // k-step 4 st
    expand_half<1>(P0, E1);
    interleave(none);
    sync();                       // stage st + 1 has landed; slot st is free
    issue(st + NS);
    read(P0, st + 1, 0);
    mma(acc, E1);                 // k-step 4 st + 1
    expand_half<0>(P1, E0);
    interleave(all);
    mma(acc, E0);                 // k-step 4 st + 2
    expand_half<1>(P1, E1);
    interleave(none);
    read(P1, st + 1, 1);
    mma(acc, E1);                 // k-step 4 st + 3
    expand_half<0>(P0, E0);
    interleave(all);
  }
  // copies of stages past the end may still be landing in LDS
  wait_vm_lgkm0<0>();
  asm volatile("" ::: "memory");

  // fast epilogue: the tile's columns inside N, 16-byte aligned output rows, 31-bit output range
  const bool fast = g.dbg_acc == nullptr && (g.ldy & 7) == 0 && (reinterpret_cast<uintptr_t>(g.y) & 15) == 0 &&
                    g.M * g.ldy * 2 < (int64_t{1} << 31) && n0 + R::BN <= g.N;
  // whole-row stores through the drained ring when rows are 16-byte aligned (uniform over
  // the workgroup, as is the barrier inside)
  static_assert(R::BM * R::BN * 2 <= L::SCALES, "the output tile fits the ring");
  if (fast) {
    __syncthreads();  // every wave's copies have landed and its last fragments are read
    ring_epilogue_staged<TM, TN, R::BM, R::BN>(g, acc, m0, n0, wm, wn, lane, scales, lds, wave, R::WAVES);
  } else if (g.swiglu) {  // element-wise stores (a third, direct-store path would cost the kernel spills)
    if constexpr (TN % 2 == 0)
      ring_epilogue_swiglu_checked<TM, TN, R::BM, R::BN>(g, acc, m0 + wm * 32, n0 + wn * 32, wm, wn, lane, scales);
  } else {
    ring_epilogue_checked<TM, TN, R::BM, R::BN>(g, acc, m0 + wm * 32, n0 + wn * 32, wm, wn, lane, scales);
  }
}

// WPE: waves per SIMD the registers must allow (2 for two 4-wave workgroups per CU).
template <GemmFamily F, bool LARGE, int WM, int WN, int TM, int TN, int NS, int WPE = 1>
hipError_t launch_ring(const GemmArgs& g, hipStream_t stream) {
  constexpr bool A8 = F == kW4A8;
  using R = Ring<WM, WN, TM, TN, NS, A8>;
  static_assert(R::BM == ring_tile(F, LARGE).bm && R::BN == ring_tile(F, LARGE).bn, "the tile the plan counts with");
  constexpr int LDS = RingLds<WM, WN, TM, TN, NS, A8>::BYTES;
  static_assert(LDS <= 160 * 1024, "LDS of one CU");
  constexpr auto kern = w4a4_gemm_ring<WM, WN, TM, TN, NS, WPE, A8>;
  const hipError_t init = set_max_lds<kern>(LDS);
  if (init != hipSuccess) return init;
  // the 31-bit operand ranges (ring_fits) bound M and N, and with them the tiles, far below a grid
  const int64_t tn = (g.N + R::BN - 1) / R::BN, tm = (g.M + R::BM - 1) / R::BM;
  return launch(kern, dim3(static_cast<unsigned>(tn * tm)), dim3(R::THREADS), LDS, stream, g.xq, g.wq, g.M, g.N,
                static_cast<int>(g.K), static_cast<int>(tm), static_cast<int>(tn * tm),
                div_magic(static_cast<uint32_t>(tm)), g);
}

// Gate/up products the entry point takes: sq.h refuses operands of about 2^31 bytes and more (one
// or two tokens with K <= 65536 are always taken, up to 16 tokens count the weights alone).  The
// slice kernel itself has no such limit.
bool swiglu_covered(const GemmArgs& g, int cus) {
  constexpr int64_t lim = int64_t{1} << 31;
  const int64_t kb = g.K / 2;
  if (g.M <= 2 && g.K <= 65536) return true;
  if (g.M <= 16) {
    const int64_t nb = 2 * ((g.N / 32 + cus - 1) / cus), skinny = g.N > 16384 ? 128 : 64;
    const int64_t past = nb <= 16 && 16 * nb < skinny ? 16 * nb : skinny;
    return (g.N + past) * kb + 64 < lim;
  }
  if (g.M <= 128) return (g.M + 128) * kb + 128 < lim && (g.N + 128) * kb + 64 < lim;
  return ring_fits(kW4A4Swiglu, g, ring_large(kW4A4Swiglu, g));
}

// Ring tiles.  At least as many 256 x 256 tiles as CUs -> those: 8 waves of 128 x 64 and four
// stages, with 8-bit codes 8 waves of 64 x 128 (8 KB of 8-bit A and 8 KB of packed B read
// from LDS per wave and stage against 16 and 4) and three stages (3 x 48 KB).  Fewer -> 128 x
// 256 tiles of 8 waves of 64 x 64, with SiLU 256 x 128 tiles of 4 waves, two per CU.
// Measured on MI355X (us, one process, interleaved), 256 x 256 against the half tiles:
//   4-bit  [2048 x 22016 x 4096] 169 vs 191   [4096 x 14336 x 4096] 427 vs 477   [4096 x 4096 x 14336] 186 vs 212
//   8-bit  [2048 x 22016 x 4096] 211 vs 255   [4096 x 28672 x 4096] 505 vs 611   [4096 x 4096 x 14336] 241 vs 290
// and with fewer than 256 large tiles the half ones: 4-bit [2048 x 4096 x 11008] 83.5 vs 123,
// 8-bit 104 vs 150.
hipError_t launch_ring_tiles(GemmFamily f, const GemmArgs& g, bool large, hipStream_t stream) {
  if (f == kW4A8)
    return large ? launch_ring<kW4A8, true, 4, 2, 2, 4, 3>(g, stream) : launch_ring<kW4A8, false, 2, 4, 2, 2, 4>(g, stream);
  if (large) return launch_ring<kW4A4, true, 2, 4, 4, 2, 4>(g, stream);
  return f == kW4A4Swiglu ? launch_ring<kW4A4Swiglu, false, 2, 2, 4, 2, 3, 2>(g, stream)
                          : launch_ring<kW4A4, false, 2, 4, 2, 2, 3>(g, stream);
}

}  // namespace

hipError_t launch_gemm(const GemmArgs& g, hipStream_t stream) {
  const GemmFamily f = g.a8 ? kW4A8 : g.swiglu ? kW4A4Swiglu : kW4A4;
  int cus = 0;
  const hipError_t e = device_cus(&cus);
  if (e != hipSuccess) return e;
  if (f == kW4A4Swiglu && !swiglu_covered(g, cus)) return hipErrorNotSupported;
  const GemmPlan p = plan_gemm(f, g, cus);
  if (p.ring_n > 0) {
    const hipError_t r = launch_ring_tiles(f, p.ring_n < g.N ? weight_rows(f, g, 0, p.ring_n) : g, p.large, stream);
    if (r != hipSuccess || p.ring_n == g.N) return r;
  }
  const GemmArgs s = weight_rows(f, g, p.ring_n, g.N);
  return f == kW4A8 ? launch_w4a8_slice(s, p.slice, stream)
                    : f == kW4A4Swiglu ? launch_w4a4_slice_swiglu(s, p.slice, stream) : launch_w4a4_slice(s, p.slice, stream);
}

}  // namespace sq
