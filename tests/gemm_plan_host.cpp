// Host side of the product's launches (csrc/gemm_plan.h) for tests/test_gemm_plan.py: no device code.
#include "gemm_plan.h"

namespace {
template <typename T>
T* at(int64_t address) {
  return reinterpret_cast<T*>(address);
}
template <typename T>
int64_t from(const T* p, int64_t base) {
  return (reinterpret_cast<int64_t>(p) - base) / static_cast<int64_t>(sizeof(T));
}
}  // namespace

// Parts of a product of family f with tiles of bm x bn: for each M, N and the element offsets of
// xq, xa, xb, wq, wa, rs, bias, y and dbg_acc (11 values); returns their count.
extern "C" int grids(int f, int64_t M, int64_t N, int64_t K, int64_t ldy, int dbg, int bm, int bn, int threads,
                     int64_t* out, int capacity) {
  constexpr int64_t base = int64_t{1} << 60;
  sq::GemmArgs g{};
  g.M = M, g.N = N, g.K = K, g.ldy = ldy, g.a8 = f == sq::kW4A8, g.swiglu = f == sq::kW4A4Swiglu;
  g.xq = at<uint8_t>(base), g.xa = at<float>(base), g.xb = at<float>(base), g.wq = at<uint8_t>(base);
  g.wa = at<float>(base), g.rs = at<int32_t>(base), g.bias = at<uint16_t>(base), g.y = at<uint16_t>(base);
  g.dbg_acc = dbg ? at<int32_t>(base) : nullptr;
  int n = 0;
  const hipError_t e = sq::in_grids(static_cast<sq::GemmFamily>(f), g, bm, bn, threads, [&](const sq::GemmArgs& p) {
    if (n == capacity) return hipErrorInvalidValue;
    const int64_t v[11] = {p.M, p.N, from(p.xq, base), from(p.xa, base), from(p.xb, base), from(p.wq, base), from(p.wa, base),
                           from(p.rs, base), from(p.bias, base), from(p.y, base), dbg ? from(p.dbg_acc, base) : -1};
    for (int i = 0; i < 11; ++i) out[11 * n + i] = v[i];
    ++n;
    return hipSuccess;
  });
  return e == hipSuccess ? n : -1;
}

// The plan of a product: ring_n, large, and the slice kernel's nb, mb, waves, ns, seg (zeros without it).
extern "C" void plan(int f, int64_t M, int64_t N, int64_t K, int dbg, int cus, int* out) {
  sq::GemmArgs g{};
  g.M = M, g.N = N, g.K = K, g.a8 = f == sq::kW4A8, g.swiglu = f == sq::kW4A4Swiglu;
  g.dbg_acc = dbg ? at<int32_t>(64) : nullptr;
  const sq::GemmPlan p = sq::plan_gemm(static_cast<sq::GemmFamily>(f), g, cus);
  const int v[7] = {static_cast<int>(p.ring_n), p.large, p.slice.nb, p.slice.mb, p.slice.ring.waves, p.slice.ring.ns, p.slice.ring.seg};
  for (int i = 0; i < 7; ++i) out[i] = v[i];
}

// The slice kernels a family is built with (nb, mb, waves, ns, seg each); returns their count.
extern "C" int built(int f, int* out) {
  int n = 0;
  for (const auto& s : sq::kSliceShape)
    for (const sq::SliceRing& r : sq::kSliceRing)
      if (sq::slice_built(static_cast<sq::GemmFamily>(f), s[0], s[1], r)) {
        const int v[5] = {s[0], s[1], r.waves, r.ns, r.seg};
        for (int i = 0; i < 5; ++i) out[5 * n + i] = v[i];
        ++n;
      }
  return n;
}
