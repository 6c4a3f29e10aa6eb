// Host-side choice between the kernels of a quantized product and of the slice kernel's tile.
#pragma once

#include <cmath>
#include <cstdint>

#include "sq_internal.h"

namespace sq {

enum GemmFamily { kW4A4 = 0, kW4A4Swiglu = 1, kW4A8 = 2 };

// How the slice kernel (gemm_slice.h) splits K: over `waves` waves, ns ring slots per wave of seg
// packed bytes per row.
struct SliceRing {
  int waves, ns, seg;
};
constexpr bool operator==(const SliceRing& a, const SliceRing& b) {
  return a.waves == b.waves && a.ns == b.ns && a.seg == b.seg;
}

// A tile of the slice kernel: 16 nb weight rows x 16 mb tokens.
struct SlicePlan {
  int nb, mb;
  SliceRing ring;
  float us;  // its estimated time
};

constexpr int kSliceShapes = 13;
constexpr int kSliceShape[kSliceShapes][2] = {{1, 1}, {2, 1}, {2, 2}, {2, 3}, {4, 2}, {4, 3}, {4, 4},
                                              {4, 5}, {4, 6}, {4, 8}, {6, 3}, {6, 4}, {8, 4}};
// Shapes a family is built with: gate and up blocks come in pairs; 8-bit codes take two
// activation bytes per weight byte, so tall tiles lose to wide ones (6 x 3, 6 x 4).
constexpr bool slice_has(GemmFamily f, int nb, int mb) {
  if (f == kW4A8) return !(nb == 2 && mb == 3) && !(nb == 4 && (mb == 5 || mb == 8));
  return nb != 6 && !(f == kW4A4Swiglu && nb == 1);
}

// Ring slots and segment length of a tile.  At most one workgroup per CU: two slots a wave,
// and 128-byte segments (whole cache lines of every row) where K leaves each wave enough of
// them.  More workgroups than CUs: one slot, so that two or three workgroups share a CU and
// cover each other's waits; there short segments take less LDS.  One-block token tiles over
// a long K are weight streams, where bytes in flight are all that counts: two long slots (one
// where K leaves a wave few segments: [1 x 4096] x [4096 x 4096] 3.6 against 3.9 us).
// Measured on MI355X (us; two slots x 128 | two x 64 | one x 128 | one x 64 bytes):
//   [77 x 28672] x [8192 x 28672], 4 x 3 blocks, 256 workgroups    32.3 | 42.1 | 47.0 | 54.6
//   [300 x 11008] x [4096 x 11008], 4 x 5, 256                     19.3 | 18.1 | 19.5 | 21.2
//   [48 x 4096] x [28672 x 4096], 4 x 3, 448                       16.2 | 14.2 | 13.8 | 13.9
//   [512 x 4096] x [22016 x 4096], 4 x 4, 2752                     -    | 57.4 | -    | 53.2
//   [16 x 8192] x [57344 x 8192], 2 x 1, 1792                      42.6 | -    | 46.4 | -
// Eight waves with one short slot each, two per SIMD, instead of four waves with two slots:
// one wave's expansion of the codes runs under the other's products.  That pays in one round
// of tiles where a wave has enough products (12 blocks) or the few stages of a short K are
// mostly start and end; over a long K whole cache lines matter more, and SiLU pairs and 8-bit
// 4 x 4 tiles gain nothing.  Time against four waves, K = 4096 | 8192 | 11008 | 14336 |
// 28672 (geometric means over 1 - 13 products each):
//   4-bit  1 x 1 .94 | - | 1.13 | 1.17 | -           2 x 2 .87 | 1.01 | 1.04 | 1.05 | 1.23
//          4 x 4 .92 | .94 | .90 | .92 | 1.13        4 x 5 .94 | .98 | .94 | .96 | 1.21
//          8 x 4 .93 | .96 | .94 | .93 | .96         4 x 2 .98 | 1.02 | 1.02 | 1.03 | 1.24
//   8-bit  2 x 1 .88 | .95 | 1.00 | 1.02 | 1.14      4 x 3 .96 | .95 | .93 | .94 | .96
//          6 x 3 .95 | .94 | .95 | .94 | 1.01        4 x 4 1.00 | 1.04 | 1.02 | 1.01 | 1.01
// ([300 x 11008] x [4096 x 11008] 4 x 5: 19.4 to 17.8 us; [24 x 4096] x [4096 x 4096] 2 x 1: 4.1
// to 3.5.)
constexpr bool slice_eight_waves(GemmFamily f, int nb, int mb, int64_t K) {
  if (f == kW4A4Swiglu || (K >= 16384 && !(f == kW4A4 && nb * mb >= 32))) return false;
  return K < 8192 || (nb * mb >= 12 && !(f == kW4A8 && nb == 4 && mb == 4));
}
// One-block tiles over a long K on few of the CUs (half; a quarter with 8-bit codes): eight waves
// with two long slots, since what bounds them is the bytes a CU has in flight (us, M = 1, four
// waves | eight; weights not in a cache): [1024 x 14336] 9.6 | 8.0, [64 x 32768] 13.4 | 9.4, [2048 x
// 28672] 16.7 | 14.2, 8-bit [1024 x 28672] 17.0 | 15.1; 8-bit on half of the CUs [16 x 14336] x [2048
// x 14336] 10.2 | 12.3, and with a tile for every CU they are even.
constexpr SliceRing slice_ring(GemmFamily f, int nb, int mb, int64_t K, bool one_round, bool few) {
  const bool a8 = f == kW4A8;
  if (few && nb == 1 && mb == 1 && K >= 8192) return {8, 2, 128};
  if (one_round && slice_eight_waves(f, nb, mb, K)) return {8, 1, 64};
  if (mb == 1 && (nb == 1 || (nb == 2 && K >= 8192))) return {4, K >= 8192 ? 2 : 1, 128};
  if (one_round)
    return {4, 2, (a8 ? nb + mb <= 4 && K >= 8192
                      : (nb + mb <= 5 && K >= 8192) || (nb + mb <= 9 && K >= 16384)) ? 128 : 64};
  return {4, 1, (nb + mb <= (a8 ? 5 : 8) && K > 4096) || (!a8 && nb + mb <= 9 && K >= 16384) ? 128 : 64};
}

// The rings a shape is built with: those slice_ring returns for it (one K of each range the rule
// tells apart).
constexpr SliceRing kSliceRing[] = {{8, 2, 128}, {8, 1, 64}, {4, 2, 128}, {4, 1, 128}, {4, 2, 64}, {4, 1, 64}};
constexpr int kSliceRings = sizeof(kSliceRing) / sizeof(kSliceRing[0]);
constexpr bool slice_built(GemmFamily f, int nb, int mb, const SliceRing& r) {
  constexpr int64_t kRanges[] = {4096, 4160, 8192, 16384};
  if (!slice_has(f, nb, mb)) return false;
  for (int64_t K : kRanges)
    for (int rounds = 0; rounds < 3; ++rounds)
      if (slice_ring(f, nb, mb, K, rounds > 0, rounds > 1) == r) return true;
  return false;
}

// Estimated times (us), fitted to 850 measured products of M = 1 .. 3600 tokens against
// weights of 2048 x 4096 to 57344 x 8192 and 8192 x 28672 on a 256-CU MI355X.  A tile costs
// its products and operand reads per 128 k, times the rounds of tiles (alone on a CU it waits
// more), next to the time the operands take from memory and from the L2s.  The tile chosen is
// 1 - 2.5 % off the best measured one on average; from 300 tokens the estimate is 5 - 7 % off
// (rms), which is why the ring below is left only for a clear gain.
// K < 4096 lies outside that fit: there the sums and stores of a tile's blocks (kBlockUs each) and
// the ring's start (kRingStartUs) are no longer hidden in the rest.  With the two terms, on 756
// products of K = 64 .. 4032 (weights not in a cache), the time is 1.6 % lower on average and 11
// instead of 29 are more than 8 % slower than on the kernels before this one: SiLU [1500 x 4096 x
// 256] 16.4 on slices, 12.2 on the ring; 8-bit [300 x 32768 x 256] 27.2 and 17.2; 4-bit [3000 x 2048
// x 2048] 25.4 and 23.0; [16 x 65536 x 128] 11.1 on 8 x 4 tiles, 8.0 on 4 x 2.
constexpr double kBlockUs = 0.05, kRingStartUs = 3.0;
constexpr bool short_k(const GemmArgs& g) { return g.K < 4096; }
// (Terms of 0.0010 sit at the fit's lower bound: those tiles cost what their operands do.)
struct SliceCost {
  float base, mem_tb, tile, ceil, alone, l2_tb;
  float shape[kSliceShapes];  // us per 128 k of a round, in the order of kSliceShape
};
inline double slice_us(GemmFamily f, const GemmArgs& g, int shape, int cus) {
  constexpr SliceCost kCost[3] = {
      {2.852f, 6.181f, 0.7274f, 0.9605f, 1.1488f, 21.85f,
       {0.0010f, 0.0117f, 0.0319f, 0.0493f, 0.0663f, 0.0963f, 0.1236f, 0.1538f, 0.1829f, 0.2423f, 0, 0, 0.2417f}},
      {3.595f, 6.706f, 0.8732f, 0.9962f, 1.2698f, 18.20f,
       {0, 0.0010f, 0.0010f, 0.0284f, 0.0470f, 0.0747f, 0.1033f, 0.1305f, 0.1636f, 0.2288f, 0, 0, 0.2280f}},
      {2.781f, 5.492f, 0.8091f, 0.8777f, 1.1424f, 21.71f,
       {0.0010f, 0.0192f, 0.0456f, 0, 0.0868f, 0.1234f, 0.1495f, 0, 0.2278f, 0, 0.1742f, 0.2252f, 0.2855f}}};
  const SliceCost& c = kCost[f];
  const int nb = kSliceShape[shape][0], mb = kSliceShape[shape][1], abytes = f == kW4A8 ? 2 : 1;
  const double M = static_cast<double>(g.M), N = static_cast<double>(g.N), K = static_cast<double>(g.K);
  const double tiles = std::ceil(M / (16 * mb)) * std::ceil(N / (16 * nb)), rounds = tiles / cus;
  double comp = (c.ceil * std::ceil(rounds) + (1 - c.ceil) * rounds) *
                (c.tile + K / 128 * c.shape[shape] + (short_k(g) ? kBlockUs * nb * mb : 0.0));
  if (rounds <= 1) comp *= c.alone;
  double mem = (N * K / 2 + M * K * abytes / 2 + (f == kW4A4Swiglu ? M * N : 2 * M * N)) / c.mem_tb * 1e-6;
  if (rounds < 1) mem /= std::sqrt(rounds);  // idle CUs stream nothing
  const double l2 = tiles * 16 * (nb + abytes * mb) * K / 2 / c.l2_tb * 1e-6;
  const double c2 = comp * comp, m2 = mem * mem, l22 = l2 * l2;
  const double us = c.base + std::sqrt(std::sqrt(c2 * c2 + m2 * m2 + l22 * l22));
  // activations far past an XCD's 4 MB of L2 (many tokens over a long K) are read again by
  // every weight tile: 17 - 29 % over the estimate where measured
  return M * K * abytes / 2 > 14e6 ? 1.25 * us : us;
}

inline SlicePlan plan_slice(GemmFamily f, const GemmArgs& g, int cus) {
  SlicePlan best{0, 0, {}, 0.0f};
  double us = 0.0;
  for (int s = 0; s < kSliceShapes; ++s) {
    const int nb = kSliceShape[s][0], mb = kSliceShape[s][1];
    if (!slice_has(f, nb, mb)) continue;
    const double t = slice_us(f, g, s, cus);
    if (best.nb == 0 || t < us) {
      best.nb = nb;
      best.mb = mb;
      us = t;
    }
  }
  best.us = static_cast<float>(us);
  const int64_t tiles = ((g.M + 16 * best.mb - 1) / (16 * best.mb)) * ((g.N + 16 * best.nb - 1) / (16 * best.nb));
  best.ring = slice_ring(f, best.nb, best.mb, g.K, tiles <= cus, (f == kW4A8 ? 4 : 2) * tiles <= cus);
  return best;
}

// Tiles of the ring kernel (w4a4_gemm.hip): 256 x 256, or half of one.
struct RingTile {
  int bm, bn;
};
constexpr RingTile ring_tile(GemmFamily f, bool large) {
  if (large) return {256, 256};
  return f == kW4A4Swiglu ? RingTile{256, 128} : RingTile{128, 256};
}
inline int64_t ring_tiles(GemmFamily f, const GemmArgs& g, bool large) {
  const RingTile t = ring_tile(f, large);
  return ((g.M + t.bm - 1) / t.bm) * ((g.N + t.bn - 1) / t.bn);
}
// The ring's 32-bit operand offsets, rows past the tiles' ends included, fit 31 bits.
inline bool ring_fits(GemmFamily f, const GemmArgs& g, bool large) {
  const RingTile t = ring_tile(f, large);
  const int64_t kb = g.K / 2, ka = f == kW4A8 ? g.K : kb;
  return (g.M + t.bm) * ka + 128 < (int64_t{1} << 31) && (g.N + t.bn) * kb + 64 < (int64_t{1} << 31);
}
// At least as many 256 x 256 tiles as the part the line was measured on has CUs.
inline bool ring_large(GemmFamily f, const GemmArgs& g) { return ring_tiles(f, g, true) >= 256; }

// Rounds of the ring kernel's tiles; the last one costs nearly as much as a full one.
inline double ring_us(GemmFamily f, const GemmArgs& g, bool large, int64_t tiles, int cus) {
  constexpr double kCost[3][2][3] = {{{4.81, 0.6454, 0.2645}, {1.03, 1.2458, 0.3400}},
                                     {{6.89, 0.6975, 0.1875}, {4.22, 1.1768, 0.3738}},
                                     {{4.81, 0.8457, 0.3277}, {7.34, 1.3151, 0.5921}}};
  const double k = static_cast<double>(g.K) / 128, rounds = static_cast<double>(tiles) / cus;
  const double* c = kCost[f][large];
  return c[0] + k * (c[1] * std::ceil(rounds) + c[2] * rounds) + (short_k(g) ? kRingStartUs : 0.0);
}

// The weight rows [r0, r1) of a product.
inline GemmArgs weight_rows(GemmFamily f, const GemmArgs& g, int64_t r0, int64_t r1) {
  GemmArgs s = g;
  s.N = r1 - r0;
  s.wq = g.wq + r0 * (g.K / 2);
  s.wa = g.wa + r0;
  s.rs = g.rs + r0;
  s.bias = g.bias ? g.bias + r0 : nullptr;
  s.y = g.y + (f == kW4A4Swiglu ? r0 / 2 : r0);
  s.dbg_acc = g.dbg_acc ? g.dbg_acc + r0 : nullptr;  // of one token: the rows keep the product's stride
  return s;
}

// The tokens [m0, m1) of a product.
inline GemmArgs token_rows(GemmFamily f, const GemmArgs& g, int64_t m0, int64_t m1) {
  GemmArgs s = g;
  s.M = m1 - m0;
  s.xq = g.xq + m0 * (f == kW4A8 ? g.K : g.K / 2);
  s.xa = g.xa + m0;
  s.xb = g.xb + m0;
  s.y = g.y + m0 * g.ldy;
  s.dbg_acc = g.dbg_acc ? g.dbg_acc + m0 * g.N : nullptr;
  return s;
}

// go(part) over the parts of a product whose tiles of bm tokens by bn weight rows fit one grid
// of `threads` a workgroup: whole tiles of tokens, and where one row of tiles is too wide, weight
// rows (of one token at a time with raw accumulators).
template <typename Go>
hipError_t in_grids(GemmFamily f, const GemmArgs& g, int bm, int bn, int threads, Go&& go) {
  const int64_t most = max_blocks(threads), tm = (g.M + bm - 1) / bm, tn = (g.N + bn - 1) / bn;
  if (tm <= most / tn) return go(g);
  if (tn > most && (g.M == 1 || !g.dbg_acc))
    return in_parts(g.N, most * bn / 64 * 64, [&](int64_t n, int64_t c) {
      return in_grids(f, weight_rows(f, g, n, n + c), bm, bn, threads, go);
    });
  return in_parts(g.M, tn > most ? 1 : most / tn * bm, [&](int64_t m, int64_t c) {
    return in_grids(f, token_rows(f, g, m, m + c), bm, bn, threads, go);
  });
}

// Kernels of a product: the ring takes weight rows [0, ring_n), the slice kernel the rest.
struct GemmPlan {
  int64_t ring_n;
  bool large;       // the ring's tiles
  SlicePlan slice;  // of the rest
};

// The slice kernel alone, the ring alone, or the ring on as many weight rows as fill whole
// rounds of its tiles and the slice kernel on the rest, where the last round would leave CUs
// idle; the ring wherever the others are not at least 7 % faster by the estimates, which is
// about their error.
// Measured on MI355X (us, three rotating weight sets, against the ring alone): W4A8 [1024 x 22016 x
// 4096] 104 vs 117 (256 tiles and 5632 rows of slices instead of two rounds for 344 tiles), [1536 x
// 22016 x 4096] 138 vs 181, [1100 x 8192 x 28672] 306 vs 446; W4A4 [2300 x 4096 x 14336] 125 vs 176,
// [2100 x 8192 x 8192] 120 vs 168; with SiLU [1300 x 22016 x 4096] 106 vs 140.
inline GemmPlan plan_gemm(GemmFamily f, const GemmArgs& g, int cus) {
  constexpr double kClear = 0.93;
  GemmPlan best{0, false, plan_slice(f, g, cus)};
  if (g.M <= 16) return best;
  double us = best.slice.us;
  const bool whole = ring_large(f, g);
  if (ring_fits(f, g, whole)) {
    const double t = ring_us(f, g, whole, ring_tiles(f, g, whole), cus);
    if (kClear * t <= us) {
      best = GemmPlan{g.N, whole, SlicePlan{}};
      us = t;
    }
  }
  if (g.dbg_acc) return best;  // its rows are the whole product's
  for (int large = 0; large < 2; ++large) {
    const RingTile t = ring_tile(f, large);
    const int64_t tm = (g.M + t.bm - 1) / t.bm, rounds = ring_tiles(f, g, large) / cus;
    const int64_t n1 = rounds * cus / tm * t.bn;
    if (n1 <= 0 || n1 >= g.N) continue;
    const GemmArgs head = weight_rows(f, g, 0, n1), tail = weight_rows(f, g, n1, g.N);
    if (!ring_fits(f, head, large)) continue;
    const SlicePlan p = plan_slice(f, tail, cus);
    const double u = ring_us(f, head, large, tm * (n1 / t.bn), cus) + p.us;
    if (u < kClear * us) {
      best = GemmPlan{n1, large != 0, p};
      us = u;
    }
  }
  return best;
}

// The slice kernel with a plan's tile.
hipError_t launch_w4a4_slice(const GemmArgs& g, const SlicePlan& p, hipStream_t stream);
hipError_t launch_w4a4_slice_swiglu(const GemmArgs& g, const SlicePlan& p, hipStream_t stream);
hipError_t launch_w4a8_slice(const GemmArgs& g, const SlicePlan& p, hipStream_t stream);

}  // namespace sq
