"""The K-sliced tile kernel of the quantized products (M up to a few hundred tokens), against
the CPU oracle: sizes that spread over the built tiles, ring depths and segment lengths, with
ragged token counts, weight rows and K (half segments, waves without a segment), biases, raw accumulators
and strided outputs.  Accumulators are exact, outputs within the fp16 output tolerance of
tests/parity.py; the vector and element-wise stores give the same bits."""

import numpy as np
import pytest
import torch

from paper_2405_16406_amd import sq

from test_gpu_parity import dev, gemm8_case, gemm_case, host, oq, say, swiglu_case, workloads

pytestmark = pytest.mark.gpu

W4A4 = [(1, 1088, 8256), (16, 60, 4160), (9, 8250, 4160), (3, 8256, 4096), (16, 8200, 8256),
        (13, 4150, 4160), (17, 16440, 4160), (18, 16448, 4096), (31, 4160, 8256), (129, 1080, 192),
        (33, 16447, 4160), (34, 16448, 4096), (255, 1088, 8256), (255, 1087, 320), (200, 4150, 4160),
        (200, 4160, 4096), (384, 1088, 16448), (16, 8252, 320), (300, 4160, 4160), (300, 4159, 4096),
        (512, 1088, 16448), (129, 4160, 192), (700, 4160, 4160), (700, 4160, 4096), (160, 4158, 320),
        (129, 22010, 192), (1000, 1088, 16448), (200, 4160, 64), (255, 8256, 192), (96, 8250, 320),
        (300, 8256, 192), (384, 4160, 320), (129, 16440, 192), (1, 16448, 320), (512, 4160, 16448),
        (384, 4160, 4160), (384, 4160, 4096), (384, 4160, 64), (1, 57344, 192), (1, 4160, 320)]

SWIGLU = [(1, 544, 8256, True), (16, 8224, 4160, True), (1, 8224, 320, False), (16, 544, 192, True),
          (17, 8224, 4160, True), (17, 4128, 192, False), (384, 544, 4160, True),
          (512, 544, 4160, False), (33, 4128, 320, True), (200, 2080, 4160, True), (1, 8224, 64, True),
          (255, 2080, 4160, True), (129, 4128, 192, False), (384, 2080, 4160, True), (160, 4128, 320, True),
          (129, 11008, 192, False), (255, 4128, 320, True), (200, 8224, 192, True), (129, 8224, 320, True),
          (5, 96, 192, True), (40, 32, 64, False), (512, 2080, 16448, True), (1000, 32, 8256, True),
          (300, 544, 8256, False), (512, 544, 16448, True), (1000, 544, 192, True)]

W4A8 = [(1, 1088, 8256), (16, 60, 4160), (9, 8250, 4160), (3, 8256, 4096), (16, 8200, 8256), (13, 4150, 192),
        (17, 16440, 4160), (18, 16448, 4096), (31, 4160, 8256), (129, 1080, 192), (16, 28730, 320),
        (16, 8252, 64), (129, 8250, 4160), (129, 4160, 192), (160, 4158, 320), (77, 28735, 192),
        (200, 8256, 320), (1, 16448, 320), (255, 8250, 320), (255, 4160, 64), (129, 16440, 192),
        (160, 8256, 320), (17, 16448, 8256), (384, 4160, 8256), (1000, 1088, 64), (65, 28730, 320),
        (1000, 4160, 192), (1, 57344, 192)]


@pytest.mark.parametrize("M,N,K", W4A4)
def test_w4a4_slice(M, N, K):
    say(f"w4a4_linear slice M={M} N={N} K={K}")
    gemm_case(M, N, K, seed=M + 3 * N + K, bias=(M + N) % 3 != 0)


@pytest.mark.parametrize("M,I,K,bias", SWIGLU)
def test_swiglu_slice(M, I, K, bias):
    say(f"w4a4_linear_swiglu slice M={M} I={I} K={K}")
    swiglu_case(M, I, K, seed=M + I + K, bias=bias)


@pytest.mark.parametrize("M,N,K", W4A8)
def test_w4a8_slice(M, N, K):
    say(f"w4a8_linear slice M={M} N={N} K={K}")
    gemm8_case(M, N, K, seed=M + 5 * N + K, bias=(M + N) % 3 != 0)


# The other tiles, wave counts, ring depths and segment lengths of the three families: four waves
# in several rounds and over a long K, eight waves elsewhere ("swiglu": rows of gate alone).
# tests/test_gemm_plan.py checks that the lists of this file reach every kernel that is built.
FORMS = [(2828, 33, 8640, "w4a4"), (98, 2952, 9536, "w4a4"), (107, 6031, 17344, "w4a4"), (169, 7901, 17216, "w4a4"),
      (1640, 1810, 192, "w4a4"), (3681, 386, 192, "w4a4"), (1, 4480, 1344, "swiglu"), (17, 4256, 1344, "swiglu"),
      (33, 4352, 2112, "swiglu"), (33, 2208, 192, "swiglu"), (1, 8352, 448, "swiglu"), (49, 3072, 16704, "swiglu"),
      (37, 8384, 576, "swiglu"), (402, 2336, 192, "swiglu"), (97, 3488, 17472, "swiglu"), (49, 4512, 192, "swiglu"),
      (92, 4192, 192, "swiglu"), (3663, 544, 192, "swiglu"), (3269, 288, 192, "swiglu"), (1, 4451, 2880, "w4a8"),
      (19, 9492, 3136, "w4a8"), (17, 6603, 8640, "w4a8"), (34, 6421, 8384, "w4a8"), (51, 9699, 8256, "w4a8"),
      (65, 12375, 192, "w4a8"), (641, 2946, 64, "w4a4"), (875, 608, 16512, "swiglu"), (558, 906, 17024, "w4a8"),
      (1822, 828, 17728, "w4a8"), (845, 1233, 16448, "w4a8"), (875, 1265, 16512, "w4a8"), (1390, 1246, 16640, "w4a8"),
      (82, 8316, 64, "w4a4"), (1986, 1554, 128, "w4a4"), (403, 160, 64, "swiglu"), (167, 2752, 64, "swiglu"),
      (880, 864, 64, "swiglu"), (1, 2048, 8192, "w4a4"), (5, 2049, 8256, "w4a4"), (16, 33, 33024, "w4a4"),
      (13, 1000, 8384, "w4a8"), (1, 2049, 8192, "w4a8")]


@pytest.mark.parametrize("M,N,K,family", FORMS)
def test_slice_forms(M, N, K, family):
    say(f"{family} slice form M={M} N={N} K={K}")
    case = dict(w4a4=gemm_case, swiglu=swiglu_case, w4a8=gemm8_case)[family]
    case(M, N, K, seed=M + N + K, sample_rows=np.unique([0, M // 2, M - 1]))


# Products that fill whole rounds of ring tiles and leave a rest for the slice kernel.  The
# accumulators' call runs as one kernel, so its outputs check the split one's bit for bit.
SPLIT = [(520, 22010, 576, False), (1000, 16448, 1088, False), (2100, 8200, 1088, False), (1300, 12288, 1088, False),
         (1000, 16448, 576, True), (2479, 3437, 1152, True), (2100, 22010, 1088, True)]
SPLIT_SWIGLU = [(1000, 8224, 1088), (2377, 1728, 1600), (2697, 1568, 1408)]
# ... and such that the ring takes whole, its last round short
WHOLE = [(2100, 8200, 576, True)]
WHOLE_SWIGLU = [(2100, 4128, 1088), (2600, 6144, 1088)]
# The ring's two tiles, ragged in M, N and K (a half stage at the end)
RING = [(2349, 1669, 448, False), (3847, 3851, 448, False), (2708, 1411, 448, True), (3883, 3841, 448, True)]
RING_SWIGLU = [(2017, 1120, 448), (3843, 1952, 448)]


@pytest.mark.parametrize("M,N,K,a8", SPLIT + WHOLE + RING)
def test_ring_and_slice(M, N, K, a8):
    say(f"ring and slice on parts of one product M={M} N={N} K={K} 8-bit={a8}")
    rows = np.array([0, 1, M // 2, M - 1])
    (gemm8_case if a8 else gemm_case)(M, N, K, seed=M + N, sample_rows=rows)


@pytest.mark.parametrize("M,I,K", SPLIT_SWIGLU + WHOLE_SWIGLU + RING_SWIGLU)
def test_ring_and_slice_swiglu(M, I, K):
    say(f"ring and slice on parts of one gate/up product M={M} I={I} K={K}")
    swiglu_case(M, I, K, seed=M + I, sample_rows=np.arange(0, M, 97))


@pytest.mark.parametrize("M,N,ld,off", [(17, 130, 131, 1), (33, 66, 70, 2), (5, 64, 64, 0), (48, 67, 72, 4)])
def test_slice_output_layouts(M, N, ld, off):
    """Row strides and offsets that take vector stores, element-wise stores and both."""
    say(f"slice output layout M={M} N={N} ld={ld} offset={off}")
    rng = workloads.rng_for(M + N)
    K = 640
    qa, qw = rng.integers(0, 16, (M, K)), rng.integers(-7, 8, (N, K))
    args = [dev(oq.pack_nibbles(qa)), dev(rng.uniform(0.1, 2, M).astype(np.float32)),
            dev(rng.uniform(-9, 0, M).astype(np.float32)), dev(oq.pack_nibbles(qw)),
            dev(rng.uniform(1e-3, 1e-2, N).astype(np.float32)), dev(qw.sum(1).astype(np.int32))]
    ref, _ = sq.w4a4_linear(*args)
    flat = torch.full((M * ld + off + 8,), float("nan"), dtype=torch.float16, device="cuda")
    view = flat[off:off + M * ld].view(M, ld)[:, :N]
    sq.w4a4_linear(*args, out=view)
    np.testing.assert_array_equal(host(view), host(ref))
    assert int(torch.isnan(flat).sum()) == flat.numel() - M * N, "bytes outside the output were written"
