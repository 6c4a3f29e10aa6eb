"""Host side of the quantized products' launches: csrc/gemm_plan.h compiled alone (no device, no GPU)."""

import ctypes
import os
import random
import subprocess

import pytest

from paper_2405_16406_amd import build

import test_gpu_slice

HERE = os.path.dirname(os.path.abspath(__file__))
W4A4, SWIGLU, W4A8 = range(3)


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("plan") / "plan.so")
    cmd = [build.hipcc(), *build.COMMON, "-O1", "-shared", os.path.join(HERE, "gemm_plan_host.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return ctypes.CDLL(out)


def plan_of(lib, family, M, N, K, dbg, cus=256):
    """(weight rows of the ring kernel, its large tiles, the slice kernel's nb, mb, waves, ns, seg)"""
    out = (ctypes.c_int * 7)()
    lib.plan(family, ctypes.c_int64(M), ctypes.c_int64(N), ctypes.c_int64(K), dbg, cus, out)
    return tuple(out)


def built(lib, family):
    out = (ctypes.c_int * 1024)()
    return {tuple(out[5 * i:5 * i + 5]) for i in range(lib.built(family, out))}


def listed(family):
    """Sizes of tests/test_gpu_slice.py that run against the oracle."""
    t = test_gpu_slice
    name = ("w4a4", "swiglu", "w4a8")[family]
    own = {W4A4: t.W4A4, SWIGLU: [c[:3] for c in t.SWIGLU], W4A8: t.W4A8}[family]
    split = t.SPLIT_SWIGLU if family == SWIGLU else [c[:3] for c in t.SPLIT if c[3] == (family == W4A8)]
    sizes = own + [c[:3] for c in t.FORMS if c[3] == name] + split
    return [(M, 2 * N if family == SWIGLU else N, K) for M, N, K in sizes]


@pytest.mark.parametrize("family", [W4A4, SWIGLU, W4A8])
def test_every_slice_kernel_is_tested(plan, family):
    """Each kernel that is built is the plan of a listed size (on 256 CUs), and every plan is built."""
    plans = [plan_of(plan, family, *c, dbg) for c in listed(family) for dbg in ((0,) if family == SWIGLU else (0, 1))]
    reached = {p[2:] for p in plans if p[2]}
    assert reached == built(plan, family)


def test_ring_sizes_run_on_the_ring(plan):
    t = test_gpu_slice
    for M, N, K, a8 in t.SPLIT:
        assert 0 < plan_of(plan, W4A8 if a8 else W4A4, M, N, K, 0)[0] < N, (M, N, K)
        assert plan_of(plan, W4A8 if a8 else W4A4, M, N, K, 1)[0] in (0, N), (M, N, K)
    for M, I, K in t.SPLIT_SWIGLU:
        assert 0 < plan_of(plan, SWIGLU, M, 2 * I, K, 0)[0] < 2 * I, (M, I, K)
    for family in (W4A4, SWIGLU, W4A8):  # half and whole 256 x 256 tiles
        sizes = [(M, 2 * I, K) for M, I, K in t.RING_SWIGLU] if family == SWIGLU else [c[:3] for c in t.RING if c[3] == (family == W4A8)]
        assert [plan_of(plan, family, *c, 0)[:2] for c in sizes] == [(c[1], i) for i, c in enumerate(sizes)]
    for M, N, K, a8 in t.WHOLE:
        assert plan_of(plan, W4A8 if a8 else W4A4, M, N, K, 0)[0] == N, (M, N, K)
    for M, I, K in t.WHOLE_SWIGLU:
        assert plan_of(plan, SWIGLU, M, 2 * I, K, 0)[0] == 2 * I, (M, I, K)


@pytest.mark.parametrize("family", [W4A4, SWIGLU, W4A8])
def test_every_plan_is_built(plan, family):
    """The tile and ring of any product are among the built kernels, on parts of other sizes too."""
    rng, forms = random.Random(family), built(plan, family)
    for _ in range(20000):
        M, N = (int(2 ** rng.uniform(0, top)) for top in (13, 17))
        K = 64 * int(2 ** rng.uniform(0, 11 if family == W4A8 else 14))
        if family == SWIGLU:
            N = max(64, N // 64 * 64)
        p = plan_of(plan, family, M, N, K, rng.randrange(2) if family != SWIGLU else 0, rng.choice([256, 256, 304, 128, 8, 1]))
        assert 0 <= p[0] <= N and (p[0] == N or p[2:] in forms), (M, N, K, p)


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


# Products of a short K, where stores and the ring's start outweigh what the estimates are fitted
# to: measured, the ring's tiles (all N) or small slices (few blocks a tile) are the faster ones.
@pytest.mark.parametrize("family,M,N,K,ring", [(SWIGLU, 1500, 4096, 256, True), (W4A8, 128, 65536, 128, True),
                                               (W4A8, 300, 32768, 256, True), (W4A4, 3000, 2048, 2048, True),
                                               (W4A4, 24, 32768, 128, False), (SWIGLU, 10, 36864, 64, False),
                                               (W4A4, 11, 29897, 64, False), (W4A8, 22, 25762, 128, False)])
def test_short_k(plan, family, M, N, K, ring):
    p = plan_of(plan, family, M, N, K, 0)
    assert p[0] == N if ring else p[0] == 0 and p[2] * p[3] <= 8, p
