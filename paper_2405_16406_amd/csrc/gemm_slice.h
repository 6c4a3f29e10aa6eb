// K-sliced tile kernel of the quantized products, from one token to a few hundred (and any
// size whose operands the prefill ring's 31-bit offsets do not cover): kernel and launcher
// templates.  gemm_plan.h chooses the tile.
#pragma once

#include "gemm_device.h"
#include "gemm_plan.h"
#include "sq_device.h"
#include "sq_internal.h"

namespace sq {

// A workgroup owns a tile of BM = 16 MB activation rows by BN = 16 NB weight rows; its W
// waves split K in segments of SEG packed bytes per row, wave w taking segments w, w + W,
// w + 2W, ...  (the W waves read W * SEG neighbouring bytes of each row at about the same
// time).  Every wave multiplies the whole tile over its segments, so a byte of either
// operand is brought into the CU once and read from LDS once, and the waves need no barrier
// until their int32 partial sums meet in LDS at the end.
//
// What bounds these sizes is the weight stream, and the chip left idle: a tile of M tokens
// by 256 weight rows gives N / 256 workgroups (16 for N = 4096), however long K is.  Small
// tiles with K split inside the workgroup give every CU work without a second pass or a
// workspace: N = 4096 and 24 tokens are 256 tiles of 16 x 32.
//   * Operands go from global memory straight into the wave's own ring slots
//     (buffer_load ... lds), SEG contiguous bytes of each of 16 rows per block, every
//     fragment is one ds_read_b128 (positions swizzled by row: no bank conflicts in 128-byte
//     rows; 64-byte rows keep some, 0.81e6 cycles against 0.32e6 LDS instructions in [300 x 11008]
//     x [4096 x 11008]), and each lane's 16 packed bytes expand into the operands of two
//     v_mfma_i32_16x16x64_i8.
//   * A stage's fragments are read into registers and its slot is refilled before the
//     products start, so every slot is in flight while the wave multiplies.
//   * Rows past M or N and bytes past K are out of the buffer ranges and land as zeros.
//   * The first copies leave as soon as a wave runs: their parameters are preloaded, the tile
//     index is divided by a multiplication, and the epilogue's scales are fetched behind them
//     (1.0 - 1.3 us less before the first products: [48 x 4096] x [28672 x 4096] with SiLU 14.0
//     to 13.2, [300 x 11008] x [4096 x 11008] 18.3 to 17.3).
// Measured on MI355X (us, three rotating weight sets, the smaller of them from the Infinity Cache;
// before: 128 x 128 and 128 x 256 ring tiles from 17 tokens, kernels of their own for fewer):
//   4-bit  [77 x 28672] x [8192 x 28672]   32.3 vs 116     [300 x 11008] x [4096 x 11008]  18.3 vs 63.4
//          [16 x 28672] x [8192 x 28672]   21.8 vs 26.8    [128 x 4096] x [4096 x 4096]     6.2 vs 21.7
//          [1 x 8192] x [57344 x 8192]     40.2 vs 43.5    [1 x 4096] x [4096 x 4096]       3.6 vs 5.4
//   8-bit  [24 x 14336] x [4096 x 14336]    9.5 vs 98.2    [8 x 8192] x [57344 x 8192]     45.4 vs 78.1
//   SiLU   [48 x 4096] x [28672 x 4096]    14.0 vs 20.7    [1 x 4096] x [22016 x 4096]      9.1 vs 11.0
// On weights of 100 MB and more, 1 to 16 tokens read 5.2 - 5.8 TB/s; smaller ones take less (1 x
// 4096 x 4096 2.3).  Where the weights come from memory, several rounds of one-slot tiles lose
// more than the ring does: [160 x 4096] x [28672 x 4096] 36.8 against 32.7, from the cache 29.5
// against 31.7.  Operands of 2 GB and more: 8 x 4 tiles against the kernel they replaced, 4-bit
// [2048 x 22016 x 4096] 230 vs 283, [4096 x 64 x 131072] 239 vs 1861; 8-bit 288 vs 413, 287 vs 1217.
template <int NB, int MB, int W, int NS, int SEG, bool A8>
struct Slice {
  static constexpr int THREADS = 64 * W;
  static constexpr int BN = 16 * NB, BM = 16 * MB;
  static constexpr int ASEG = A8 ? 2 * SEG : SEG;  // activation bytes per row and segment
  static constexpr int WCP = SEG / 64;             // 1 KB copies per 16-row block: weights
  static constexpr int ACP = ASEG / 64;            // activations
  static constexpr int OPS = NB * WCP + MB * ACP;  // copies per stage of a wave
  static constexpr int STAGE = OPS * 1024;
  static constexpr int RING = W * NS * STAGE;
  static constexpr int XPS = SEG / 64;             // chunk columns (two k-steps each) per stage
  // partial sums: PASS blocks of every wave at a time, in the drained ring (an even number,
  // so that a gate block and its up block meet in one pass)
  static constexpr int FIT = NS * OPS;
  static constexpr int PASS = FIT < NB * MB ? FIT / 2 * 2 : NB * MB;
  static constexpr int SCALES = 2 * BM + 3 * BN;   // floats, after the ring
  static constexpr int LDS = RING + SCALES * 4;
  static_assert((NS - 1) * OPS <= 63, "outstanding copies fit the vmcnt counter");
  static_assert(PASS >= 1 && PASS * W * 1024 <= RING, "partial sums fit the ring");
  static_assert(LDS <= 160 * 1024, "LDS of one CU");
};

// Position of 16-byte chunk c of row r (of 16) in a block whose rows are RB bytes, so that the 16
// lanes of one chunk column fall on distinct banks.
template <int RB>
__device__ __forceinline__ uint32_t slice_pos(int r, int c) {
  constexpr int SH = RB == 64 ? 2 : RB == 128 ? 1 : 0;
  return static_cast<uint32_t>(c ^ ((r >> SH) & (RB / 16 - 1)));
}

template <int NB, int MB, int W, int NS, int SEG, bool A8, bool SW>
__global__ void __launch_bounds__(64 * W, 2)
w4_gemm_slice(const uint8_t* xq, const uint8_t* wq, int64_t M, int64_t N, int K, int tiles_m, int total, uint32_t magic,
              GemmArgs g) {
  g.xq = xq;
  g.wq = wq;
  g.M = M;
  g.N = N;
  g.K = K;
  using S = Slice<NB, MB, W, NS, SEG, A8>;
  static_assert(!SW || NB % 2 == 0, "gate/up block pairs");
  extern __shared__ __attribute__((aligned(16))) uint8_t lds[];
  float* const scales = reinterpret_cast<float*>(lds + S::RING);  // rowA, rowB [BM], colS, colR, colB [BN]
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int r = lane & 15, sg = lane >> 4;
  const uint32_t KB = static_cast<uint32_t>(g.K / 2);
  const uint32_t XB = A8 ? 2 * KB : KB;  // activation bytes per row

  // tile: workgroups go round-robin over the 8 XCDs; each XCD takes a contiguous range of
  // tiles, M fastest, so the M tiles of a weight tile share its L2
  const int bid = static_cast<int>(blockIdx.x);
  const int q8 = total / 8, r8 = total % 8, xcd = bid % 8, idx = bid / 8;
  const int tile = xcd < r8 ? xcd * (q8 + 1) + idx : r8 * (q8 + 1) + (xcd - r8) * q8 + idx;
  uint32_t tq, tr;
  div_rem(tile, tiles_m, magic, tq, tr);
  const int64_t m0 = static_cast<int64_t>(tr) * S::BM;
  const int64_t nt = tq;
  // weight row of local block j relative to nbase: consecutive blocks, or with SW pairs of a
  // gate block (2 i) and its up block (2 i + 1)
  const int64_t pair0 = nt * (NB / 2);
  const int64_t nbase = SW ? 64 * (pair0 / 2) : nt * S::BN;
  auto block_row = [&](int j) -> int {
    if constexpr (SW) {
      const int p = static_cast<int>(pair0 % 2) + j / 2;  // pair counted from the even one at nbase
      return 64 * (p / 2) + 16 * (p % 2) + 32 * (j % 2);
    } else {
      return 16 * j;
    }
  };

  // buffers relative to the tile; rows past M or N and bytes past K are out of range: zeros
  const int64_t rows_m = g.M - m0 < S::BM ? g.M - m0 : S::BM;
  const int64_t span_n = SW ? 2 * S::BN + 64 : S::BN;
  const int64_t rows_n = g.N - nbase < span_n ? g.N - nbase : span_n;
  const __amdgpu_buffer_rsrc_t rsa = buf_rsrc(g.xq + m0 * XB, rows_m * XB);
  const __amdgpu_buffer_rsrc_t rsb = buf_rsrc(g.wq + nbase * KB, rows_n * KB);
  uint8_t* const ring = lds + w * NS * S::STAGE;
  const int nseg = static_cast<int>((KB + SEG - 1) / SEG);
  const int T = (nseg + W - 1) / W;  // stages of a wave (the last may lie past K: zeros)

  // copy q of a block: lane i brings row q RPI + i / LPR, the chunk that belongs at its
  // landing position
  constexpr int WL = SEG / 16, AL = S::ASEG / 16;  // lanes per row
  uint32_t wrow[S::WCP], wcol[S::WCP], arow[S::ACP], acol[S::ACP];
#pragma unroll
  for (int q = 0; q < S::WCP; ++q) {
    const int rr = q * (64 / WL) + lane / WL;
    wcol[q] = 16 * slice_pos<SEG>(rr, lane % WL);
    wrow[q] = static_cast<uint32_t>(rr) * KB;
  }
#pragma unroll
  for (int q = 0; q < S::ACP; ++q) {
    const int rr = q * (64 / AL) + lane / AL;
    acol[q] = 16 * slice_pos<S::ASEG>(rr, lane % AL);
    arow[q] = static_cast<uint32_t>(rr) * XB;
  }
  uint32_t boff[NB];
#pragma unroll
  for (int j = 0; j < NB; ++j) boff[j] = static_cast<uint32_t>(block_row(j)) * KB;

  auto issue = [&](auto slot_c, int t) {
    constexpr int slot = decltype(slot_c)::value;
    // the slot's previous reads must have returned before a copy may land in it
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    asm volatile("" ::: "memory");
    const uint32_t seg = static_cast<uint32_t>(t) * W + w;
    const uint32_t k0 = t < T ? seg * SEG : KB;  // past the run: nothing in range
    uint8_t* const sb = ring + slot * S::STAGE;
#pragma unroll
    for (int q = 0; q < S::WCP; ++q) {
      const uint32_t k = k0 + wcol[q];
      const uint32_t o = k < KB ? wrow[q] + k : 0x80000000u;
#pragma unroll
      for (int j = 0; j < NB; ++j) {
        auto* dst = reinterpret_cast<__attribute__((address_space(3))) void*>(
            reinterpret_cast<uintptr_t>(sb + (j * S::WCP + q) * 1024));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsb, dst, 16, static_cast<int>(o + boff[j]), 0, 0, 0);
      }
    }
#pragma unroll
    for (int q = 0; q < S::ACP; ++q) {
      const uint32_t k = (A8 ? 2 * k0 : k0) + acol[q];
      const uint32_t o = k < XB ? arow[q] + k : 0x80000000u;
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        auto* dst = reinterpret_cast<__attribute__((address_space(3))) void*>(
            reinterpret_cast<uintptr_t>(sb + (NB * S::WCP + i * S::ACP + q) * 1024));
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsa, dst, 16, static_cast<int>(o + static_cast<uint32_t>(16 * i) * XB), 0, 0, 0);
      }
    }
  };

  v4i acc[NB][MB];
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < MB; ++i) acc[j][i] = v4i{0, 0, 0, 0};

  issue(std::integral_constant<int, 0>{}, 0);
  // epilogue scales: fetched behind the first stage's copies (clamped indices, no branch around
  // a load).  Small tiles, and eight waves (one workgroup per CU in any case), stage them after
  // the products, off the first stage's path (4 x 3 tiles, [48 x 4096] x [28672 x 4096] with SiLU:
  // 13.2 against 13.7 us; 4 x 5, [300 x 11008] x [4096 x 11008]: 17.4 against 18.9); larger ones
  // of four waves when that stage has landed, since held through the products they cost a
  // workgroup per CU ([320 x 8192] x [57344 x 8192]: 167 against 180).
  constexpr bool kLate = NB * MB <= 12 || W == 8;
  constexpr int SPT = (S::SCALES + S::THREADS - 1) / S::THREADS;
  float fxa[SPT], fxb[SPT], fwa[SPT];
  int32_t frs[SPT];
  uint16_t fbi[SPT];
  auto col_of = [&](int t) -> int64_t { return nbase + block_row(t / 16) + t % 16; };
  const uint16_t* const bp = g.bias ? g.bias : reinterpret_cast<const uint16_t*>(g.wa);
#pragma unroll
  for (int u = 0; u < SPT; ++u) {
    const int x = static_cast<int>(threadIdx.x) + u * S::THREADS;
    const int t = x < 2 * S::BM ? 0 : x - 2 * S::BM;
    const int64_t m = m0 + x % S::BM, n = col_of(t % S::BN);
    const int64_t mc = m < g.M ? m : g.M - 1, nc = n < g.N ? n : g.N - 1;
    fxa[u] = g.xa[mc];
    fxb[u] = g.xb[mc];
    fwa[u] = g.wa[nc];
    frs[u] = g.rs[nc];
    fbi[u] = bp[nc];
  }
  static_for<NS - 1>([&](auto pc) { issue(std::integral_constant<int, decltype(pc)::value + 1>{}, decltype(pc)::value + 1); });

  auto stage_scales = [&] {
#pragma unroll
    for (int u = 0; u < SPT; ++u) {
      const int x = static_cast<int>(threadIdx.x) + u * S::THREADS;
      const int t = x < 2 * S::BM ? 0 : x - 2 * S::BM;
      const bool mok = m0 + x % S::BM < g.M, nok = col_of(t % S::BN) < g.N;
      float v;
      if (x < S::BM)
        v = mok ? __fmul_rn(fxa[u], 0.0625f) : 0.0f;
      else if (x < 2 * S::BM)
        v = mok ? (A8 ? __fmaf_rn(128.0f, fxa[u], fxb[u]) : fxb[u]) : 0.0f;
      else if (t < S::BN)
        v = nok ? fwa[u] : 0.0f;
      else if (t < 2 * S::BN)
        v = nok ? static_cast<float>(frs[u]) : 0.0f;
      else
        v = nok && g.bias ? h2f(fbi[u]) : 0.0f;
      if (x < S::SCALES) scales[x] = v;
    }
  };
  if constexpr (!kLate) stage_scales();

  for (int t0 = 0; t0 < T; t0 += NS) {
    static_for<NS>([&](auto pc) {
      constexpr int p = decltype(pc)::value;
      if (t0 + p < T) {  // uniform over the workgroup
        wait_vm_lgkm0<(NS - 1) * S::OPS>();  // stage t0 + p has landed
        asm volatile("" ::: "memory");
        // the stage's fragments go to registers and its slot takes the next copy before the
        // products start: every slot is in flight while the wave multiplies
        const uint8_t* const sb = ring + p * S::STAGE;
        v4u wv[S::XPS][NB], av[S::XPS][MB][A8 ? 2 : 1];
#pragma unroll
        for (int x = 0; x < S::XPS; ++x) {
          const int c = 4 * x + sg;  // the lane's weight chunk of the segment: 32 codes
#pragma unroll
          for (int j = 0; j < NB; ++j)
            wv[x][j] = *reinterpret_cast<const v4u*>(sb + j * S::WCP * 1024 + r * SEG + 16 * slice_pos<SEG>(r, c));
#pragma unroll
          for (int i = 0; i < MB; ++i) {
            const uint8_t* ab = sb + (NB * S::WCP + i * S::ACP) * 1024 + r * S::ASEG;
            if constexpr (A8) {
              av[x][i][0] = *reinterpret_cast<const v4u*>(ab + 16 * slice_pos<S::ASEG>(r, 2 * c));
              av[x][i][1] = *reinterpret_cast<const v4u*>(ab + 16 * slice_pos<S::ASEG>(r, 2 * c + 1));
            } else {
              av[x][i][0] = *reinterpret_cast<const v4u*>(ab + 16 * slice_pos<S::ASEG>(r, c));
            }
          }
        }
        issue(pc, t0 + p + NS);
#pragma unroll
        for (int x = 0; x < S::XPS; ++x) {
#pragma unroll
          for (int hh = 0; hh < 2; ++hh) {
            v4i ea[MB], eb[NB];
#pragma unroll
            for (int j = 0; j < NB; ++j) {
              const uint32_t b0 = wv[x][j][2 * hh], b1 = wv[x][j][2 * hh + 1];
              eb[j] = v4i{static_cast<int>((b0 << 4) & 0xF0F0F0F0u), static_cast<int>(b0 & 0xF0F0F0F0u),
                          static_cast<int>((b1 << 4) & 0xF0F0F0F0u), static_cast<int>(b1 & 0xF0F0F0F0u)};
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) {
              if constexpr (A8) {
                ea[i] = act8_operand(av[x][i][hh]);
              } else {
                const uint32_t a0 = av[x][i][0][2 * hh], a1 = av[x][i][0][2 * hh + 1];
                ea[i] = v4i{static_cast<int>(a0 & 0x0F0F0F0Fu), static_cast<int>((a0 >> 4) & 0x0F0F0F0Fu),
                            static_cast<int>(a1 & 0x0F0F0F0Fu), static_cast<int>((a1 >> 4) & 0x0F0F0F0Fu)};
              }
            }
#pragma unroll
            for (int i = 0; i < MB; ++i)
#pragma unroll
              for (int j = 0; j < NB; ++j)
                acc[j][i] = __builtin_amdgcn_mfma_i32_16x16x64_i8(eb[j], ea[i], acc[j][i], 0, 0, 0);
          }
        }
      }
    });
  }
  if constexpr (kLate) stage_scales();
  wait_vm_lgkm0<0>();  // copies past the run (zeros) have landed
  __syncthreads();     // every wave is done with its ring; the scales are in place

  // The weights are the MFMA A operand: lane r + 16 sg holds output row m = r of the block,
  // columns 4 sg .. 4 sg + 3.  Blocks in order j fastest; wave w finishes units w, w + W, ...
  const float* const rowA = scales;
  const float* const rowB = rowA + S::BM;
  const float* const colS = rowB + S::BM;
  const float* const colR = colS + S::BN;
  const float* const colB = colR + S::BN;
  v4i* const part = reinterpret_cast<v4i*>(lds);  // [wave][PASS][lane]
  constexpr int TOT = NB * MB, U = SW ? 2 : 1;
  static_for<(TOT + S::PASS - 1) / S::PASS>([&](auto qc) {
    constexpr int b0 = decltype(qc)::value * S::PASS;
    constexpr int nblk = TOT - b0 < S::PASS ? TOT - b0 : S::PASS;
    if constexpr (b0 > 0) __syncthreads();
    static_for<nblk>([&](auto bc) {
      constexpr int b = b0 + decltype(bc)::value;
      part[(w * S::PASS + b - b0) * 64 + lane] = acc[b % NB][b / NB];
    });
    __syncthreads();
    for (int u = w; u < nblk / U; u += W) {
      const int b = b0 + u * U;
      const int j = b % NB, i = b / NB;
      v4i s0 = part[(u * U) * 64 + lane], s1 = {0, 0, 0, 0};
      if constexpr (SW) s1 = part[(u * U + 1) * 64 + lane];
#pragma unroll
      for (int v = 1; v < W; ++v) {
        s0 += part[(v * S::PASS + u * U) * 64 + lane];
        if constexpr (SW) s1 += part[(v * S::PASS + u * U + 1) * 64 + lane];
      }
      const int64_t m = m0 + 16 * i + r;
      const float ra = rowA[16 * i + r], rb = rowB[16 * i + r];
      const int c0 = 16 * j + 4 * sg;
      float yv[4];
      int64_t n, nlim;
      if constexpr (SW) {
        const int c1 = c0 + 16;
        const int64_t p = pair0 + j / 2;
        n = 32 * (p / 2) + 16 * (p % 2) + 4 * sg;
        nlim = g.N / 2;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float gv = fp32_result(__fmaf_rn(ra, __fmul_rn(colS[c0 + e], static_cast<float>(s0[e])),
                                                 __fmaf_rn(rb, __fmul_rn(colS[c0 + e], colR[c0 + e]), colB[c0 + e])));
          const float uv = fp32_result(__fmaf_rn(ra, __fmul_rn(colS[c1 + e], static_cast<float>(s1[e])),
                                                 __fmaf_rn(rb, __fmul_rn(colS[c1 + e], colR[c1 + e]), colB[c1 + e])));
          yv[e] = fp32_result(swiglu_value(gv, uv));
        }
      } else {
        n = nbase + c0;
        nlim = g.N;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          yv[e] = fp32_result(__fmaf_rn(ra, __fmul_rn(colS[c0 + e], static_cast<float>(s0[e])),
                                        __fmaf_rn(rb, __fmul_rn(colS[c0 + e], colR[c0 + e]), colB[c0 + e])));
      }
      if (m >= g.M) continue;
      uint16_t* const yp = g.y + m * g.ldy + n;
      if (n + 3 < nlim && (reinterpret_cast<uintptr_t>(yp) & 7) == 0) {
        *reinterpret_cast<v2u*>(yp) = v2u{f2h2(yv[0], yv[1]), f2h2(yv[2], yv[3])};
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (n + e < nlim) yp[e] = f2h(yv[e]);
      }
      if constexpr (!SW) {
        if (g.dbg_acc) {
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (n + e < nlim) g.dbg_acc[m * g.N + n + e] = (s0[e] >> 4) + (A8 ? 128 * g.rs[n + e] : 0);
        }
      }
    }
  });
}

template <int NB, int MB, int W, int NS, int SEG, GemmFamily F>
hipError_t launch_slice(const GemmArgs& g, hipStream_t stream) {
  constexpr bool A8 = F == kW4A8, SW = F == kW4A4Swiglu;
  using S = Slice<NB, MB, W, NS, SEG, A8>;
  constexpr auto kern = w4_gemm_slice<NB, MB, W, NS, SEG, A8, SW>;
  const hipError_t init = set_max_lds<kern>(S::LDS);
  if (init != hipSuccess) return init;
  return in_grids(F, g, S::BM, S::BN, S::THREADS, [stream](const GemmArgs& p) {
    const int64_t tn = (p.N + S::BN - 1) / S::BN, tm = (p.M + S::BM - 1) / S::BM;
    return launch(kern, dim3(static_cast<unsigned>(tn * tm)), dim3(S::THREADS), S::LDS, stream, p.xq, p.wq, p.M, p.N,
                  static_cast<int>(p.K), static_cast<int>(tm), static_cast<int>(tn * tm),
                  div_magic(static_cast<uint32_t>(tm)), p);
  });
}

// The plan's kernel, of those slice_ring can ask for.
template <GemmFamily F>
hipError_t launch_slice_plan(const GemmArgs& g, const SlicePlan& p, hipStream_t stream) {
  hipError_t e = hipErrorInvalidValue;
  static_for<kSliceShapes * kSliceRings>([&](auto ic) {
    constexpr int i = decltype(ic)::value;
    constexpr int nb = kSliceShape[i / kSliceRings][0], mb = kSliceShape[i / kSliceRings][1];
    constexpr SliceRing r = kSliceRing[i % kSliceRings];
    if constexpr (slice_built(F, nb, mb, r))
      if (p.nb == nb && p.mb == mb && p.ring == r) e = launch_slice<nb, mb, r.waves, r.ns, r.seg, F>(g, stream);
  });
  return e;
}

}  // namespace sq
