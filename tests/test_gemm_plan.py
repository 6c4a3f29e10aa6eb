"""Host side of the quantized products' launches: csrc/gemm_plan.h compiled alone (no device, no GPU)."""

import ctypes
import os
import subprocess

import pytest

from paper_2405_16406_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
W4A4, SWIGLU, W4A8 = range(3)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plan") / "plan.so")
    cmd = [build.hipcc(), *build.COMMON, "-O1", "-shared", os.path.join(HERE, "gemm_plan_host.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(out)


# Products of more workgroups than one grid holds (2^32 threads), and their neighbours that fit.
@pytest.mark.parametrize("family,M,N,K,bm,bn,threads", [
    (W4A4, (1 << 30) + 5, 72, 64, 64, 128, 256), (W4A4, (1 << 30) - 64, 72, 64, 64, 128, 256), (W4A4, (1 << 31) - 1, 8, 64, 128, 64, 256),
    (W4A4, 1 << 26, 2048, 64, 128, 64, 256), (W4A4, 1, (1 << 31) - 1, 64, 64, 128, 256), (W4A4, 2, (1 << 31) - 1, 64, 64, 128, 256),
    (W4A8, (1 << 29) + 77, 130, 128, 32, 64, 256), (W4A8, 5, 1 << 30, 64, 16, 16, 512), (SWIGLU, (1 << 29) + 1, 192, 64, 64, 128, 256),
    (SWIGLU, 3, (1 << 31) - 64, 64, 16, 32, 256), (W4A4, 300, 4096, 11008, 80, 64, 512)])
def test_products_past_one_grid(plan, family, M, N, K, bm, bn, threads):
    """The parts cover the product once, each within a grid, with every operand at its place."""
    for dbg in (0,) if family == SWIGLU else (0, 1):  # no raw accumulators with SiLU
        check_parts(plan, family, M, N, K, bm, bn, threads, dbg)


def check_parts(plan, family, M, N, K, bm, bn, threads, dbg):
    cols = N // 2 if family == SWIGLU else N
    ldy = cols + 3
    buf = (ctypes.c_int64 * (11 * 8192))()
    i64 = ctypes.c_int64
    n = plan.grids(family, i64(M), i64(N), i64(K), i64(ldy), dbg, bm, bn, threads, buf, 8192)
    assert n >= 1
    area, seen = 0, []
    for i in range(n):
        m_, n_, xq, xa, xb, wq, wa, rs, bias, y, acc = buf[11 * i:11 * i + 11]
        assert -(-m_ // bm) * -(-n_ // bn) * threads < 1 << 32
        m0, n0 = xa, wa
        assert xb == m0 and rs == n0 and bias == n0
        assert xq == m0 * (K if family == W4A8 else K // 2) and wq == n0 * (K // 2)
        assert y == m0 * ldy + (n0 // 2 if family == SWIGLU else n0)
        if family == SWIGLU:
            assert n0 % 64 == 0 and n_ % 64 == 0
        if dbg:  # a part's rows keep the product's stride only where it has whole rows, or one
            assert acc == m0 * N + n0 and (n_ == N or m_ == 1)
        assert m0 + m_ <= M and n0 + n_ <= N
        seen.append((m0, n0, m_, n_))
        area += m_ * n_
    assert area == M * N and len({s[:2] for s in seen}) == n
    if -(-M // bm) * -(-N // bn) * threads < 1 << 32:
        assert n == 1
