"""The K-sliced tile kernel of the quantized products (M up to a few hundred tokens), against
the CPU oracle: one case per built tile, ring depth and segment length, with ragged token
counts, weight rows and K (half segments, waves without a segment), biases, raw accumulators
and strided outputs.  Accumulators are exact, outputs within the fp16 output tolerance of
tests/parity.py; the vector and element-wise stores give the same bits."""

import numpy as np
import pytest
import torch

from paper_2405_16406_amd import sq

from test_gpu_parity import dev, gemm8_case, gemm_case, host, oq, say, swiglu_case, workloads

pytestmark = pytest.mark.gpu

# token counts at the tiles' edges (16 nb x 16 mb blocks, ns slots of seg bytes in the comments)
W4A4 = [(1, 1088, 8256),    # 1 x 1, 2 x 128
        (16, 60, 4160),     # 1 x 1, 2 x 64; the last block of weight rows ragged
        (9, 8250, 4160),    # 2 x 1, 1 x 128
        (3, 8256, 4096),    # 2 x 1, 1 x 64
        (16, 8200, 8256),   # 2 x 1, 2 x 128
        (13, 4150, 4160),   # 2 x 1, 2 x 64
        (17, 16440, 4160),  # 2 x 2, 1 x 128
        (18, 16448, 4096),  # 2 x 2, 1 x 64
        (31, 4160, 8256),   # 2 x 2, 2 x 128
        (129, 1080, 192),   # 2 x 2, 2 x 64
        (33, 16447, 4160),  # 2 x 3, 1 x 128
        (34, 16448, 4096),  # 2 x 3, 1 x 64
        (255, 1088, 8256),  # 2 x 3, 2 x 128
        (255, 1087, 320),   # 2 x 3, 2 x 64
        (200, 4150, 4160),  # 4 x 2, 1 x 128
        (200, 4160, 4096),  # 4 x 2, 1 x 64
        (384, 1088, 16448),  # 4 x 2, 2 x 128
        (16, 8252, 320),    # 4 x 2, 2 x 64
        (300, 4160, 4160),  # 4 x 3, 1 x 128
        (300, 4159, 4096),  # 4 x 3, 1 x 64
        (512, 1088, 16448),  # 4 x 3, 2 x 128
        (129, 4160, 192),   # 4 x 3, 2 x 64
        (700, 4160, 4160),  # 4 x 4, 1 x 128
        (700, 4160, 4096),  # 4 x 4, 1 x 64
        (160, 4158, 320),   # 4 x 4, 2 x 64
        (129, 22010, 192),  # 4 x 5, 1 x 64
        (1000, 1088, 16448),  # 4 x 5, 2 x 128
        (200, 4160, 64),    # 4 x 5, 2 x 64: one segment, three waves without any
        (255, 8256, 192),   # 4 x 6, 1 x 64
        (96, 8250, 320),    # 4 x 6, 2 x 64
        (300, 8256, 192),   # 4 x 8, 1 x 64
        (384, 4160, 320),   # 4 x 8, 2 x 64
        (129, 16440, 192),  # 8 x 4, 1 x 64
        (1, 16448, 320)]    # 8 x 4, 2 x 64

SWIGLU = [(1, 544, 8256, True), (16, 8224, 4160, True), (1, 8224, 320, False), (16, 544, 192, True),
          (17, 8224, 4160, True), (17, 4128, 192, False), (384, 544, 4160, True),
          (512, 544, 4160, False), (33, 4128, 320, True), (200, 2080, 4160, True), (1, 8224, 64, True),
          (255, 2080, 4160, True), (129, 4128, 192, False), (384, 2080, 4160, True), (160, 4128, 320, True),
          (129, 11008, 192, False), (255, 4128, 320, True), (200, 8224, 192, True), (129, 8224, 320, True),
          (5, 96, 192, True), (40, 32, 64, False)]

W4A8 = [(1, 1088, 8256), (16, 60, 4160), (9, 8250, 4160), (3, 8256, 4096), (16, 8200, 8256), (13, 4150, 192),
        (17, 16440, 4160), (18, 16448, 4096), (31, 4160, 8256), (129, 1080, 192), (16, 28730, 320),
        (16, 8252, 64), (129, 8250, 4160), (129, 4160, 192), (160, 4158, 320), (77, 28735, 192),
        (200, 8256, 320), (1, 16448, 320), (255, 8250, 320), (255, 4160, 64), (129, 16440, 192),
        (160, 8256, 320)]


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
