// Host-side choice between the kernels of a quantized product and of the slice kernel's tile.
#pragma once

#include <cmath>
#include <cstdint>

#include "sq_internal.h"

namespace sq {

enum GemmFamily { kW4A4 = 0, kW4A4Swiglu = 1, kW4A8 = 2 };

// A tile of the slice kernel (gemm_slice.h): 16 nb weight rows x 16 mb tokens, ns ring slots
// per wave of seg packed bytes per row.
struct SlicePlan {
  int nb, mb, ns, seg;
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
// a long K are weight streams, where bytes in flight are all that counts: two long slots.
// Measured on MI355X (us; two slots x 128 | two x 64 | one x 128 | one x 64 bytes):
//   [77 x 28672] x [8192 x 28672], 4 x 3 blocks, 256 workgroups    32.3 | 42.1 | 47.0 | 54.6
//   [300 x 11008] x [4096 x 11008], 4 x 5, 256                     19.3 | 18.1 | 19.5 | 21.2
//   [48 x 4096] x [28672 x 4096], 4 x 3, 448                       16.2 | 14.2 | 13.8 | 13.9
//   [512 x 4096] x [22016 x 4096], 4 x 4, 2752                     -    | 57.4 | -    | 53.2
//   [16 x 8192] x [57344 x 8192], 2 x 1, 1792                      42.6 | -    | 46.4 | -
inline void slice_ring(GemmFamily f, int nb, int mb, int64_t K, bool one_round, int* ns, int* seg) {
  const bool a8 = f == kW4A8;
  if (mb == 1 && nb <= 2 && K >= 8192) {
    *ns = 2;
    *seg = 128;
  } else if (one_round) {
    *ns = 2;
    *seg = (a8 ? nb + mb <= 4 && K >= 8192
               : (nb + mb <= 5 && K >= 8192) || (nb + mb <= 9 && K >= 16384)) ? 128 : 64;
  } else {
    *ns = 1;
    *seg = nb + mb <= (a8 ? 5 : 8) && K > 4096 ? 128 : 64;
  }
}

// Estimated times (us), fitted to 495 measured products of M = 1 .. 1400 tokens against
// weights of 4096 x 4096 to 57344 x 8192 and 8192 x 28672 on a 256-CU MI355X: the chosen tile
// is 1.0 - 2.5 % off the best measured one on average, and the choice between slice and ring
// below 0.1 - 0.2 %.  A tile costs its products and its operand reads per 128 k, times the
// workgroups of the busiest CU (alone on a CU it waits more), next to the time the operands
// take from memory.
struct SliceCost {
  double tile, prod, oper, base, rate, alone;
};
inline double slice_us(GemmFamily f, const GemmArgs& g, int nb, int mb, int cus) {
  constexpr SliceCost kCost[3] = {{0.297, 0.00609, 0.00481, 3.517, 4.153, 1.048},
                                  {0.171, 0.00675, 0.00360, 2.805, 3.578, 1.942},
                                  {0.117, 0.00663, 0.00516, 4.395, 3.888, 1.001}};
  const SliceCost& c = kCost[f];
  const double M = static_cast<double>(g.M), N = static_cast<double>(g.N), K = static_cast<double>(g.K);
  const int abytes = f == kW4A8 ? 2 : 1;
  const double tiles = std::ceil(M / (16 * mb)) * std::ceil(N / (16 * nb));
  const double busy = std::ceil(tiles / cus);
  double comp = busy * (c.tile + K / 128 * (c.prod * nb * mb + c.oper * (nb + abytes * mb)));
  if (busy == 1) comp *= c.alone;
  const double mem = (N * K / 2 + M * K * abytes / 2 + 2 * M * N) / c.rate * 1e-6;
  const double c2 = comp * comp, m2 = mem * mem;
  return c.base + std::sqrt(std::sqrt(c2 * c2 + m2 * m2));
}

inline SlicePlan plan_slice(GemmFamily f, const GemmArgs& g, int cus) {
  SlicePlan best{0, 0, 0, 0, 0.0f};
  double us = 0.0;
  for (int s = 0; s < kSliceShapes; ++s) {
    const int nb = kSliceShape[s][0], mb = kSliceShape[s][1];
    if (!slice_has(f, nb, mb)) continue;
    const double t = slice_us(f, g, nb, mb, cus);
    if (best.nb == 0 || t < us) {
      best.nb = nb;
      best.mb = mb;
      us = t;
    }
  }
  best.us = static_cast<float>(us);
  const int64_t tiles = ((g.M + 16 * best.mb - 1) / (16 * best.mb)) * ((g.N + 16 * best.nb - 1) / (16 * best.nb));
  slice_ring(f, best.nb, best.mb, g.K, tiles <= cus, &best.ns, &best.seg);
  return best;
}

// Rounds of the ring kernel's tiles (256 x 256 from one per CU on, else half as large): the
// last one costs as much as a full one.
inline double ring_us(GemmFamily f, const GemmArgs& g, int cus) {
  constexpr double kCost[3][2][3] = {{{4.81, 0.6454, 0.2645}, {1.03, 1.2458, 0.3400}},
                                     {{6.89, 0.6975, 0.1875}, {4.22, 1.1768, 0.3738}},
                                     {{4.81, 0.8457, 0.3277}, {7.34, 1.3151, 0.5921}}};
  const int64_t big = ((g.M + 255) / 256) * ((g.N + 255) / 256);
  const bool large = big >= 256;
  const int64_t half = f == kW4A4Swiglu ? ((g.M + 255) / 256) * ((g.N + 127) / 128)
                                        : ((g.M + 127) / 128) * ((g.N + 255) / 256);
  const double tiles = static_cast<double>(large ? big : half), k = static_cast<double>(g.K) / 128;
  const double* c = kCost[f][large];
  return c[0] + k * (c[1] * std::ceil(tiles / cus) + c[2] * tiles / cus);
}

// The slice kernel with a plan's tile.
hipError_t launch_w4a4_slice(const GemmArgs& g, const SlicePlan& p, hipStream_t stream);
hipError_t launch_w4a4_slice_swiglu(const GemmArgs& g, const SlicePlan& p, hipStream_t stream);
hipError_t launch_w4a8_slice(const GemmArgs& g, const SlicePlan& p, hipStream_t stream);

}  // namespace sq
