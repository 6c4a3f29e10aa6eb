"""Weight packing on the matrix-core rotation kernels and the register kernel, against the CPU
oracle: the rotations the library has fast kernels for, with row counts around the kernels' row
sets and grids, strided and sign-flipped rows, and degenerate rows."""

import numpy as np
import pytest
import torch

from oracle import hadamard as ohad
from oracle import linear as olin
from paper_2405_16406_amd import sq, workloads

import parity
from test_gpu_parity import check_w, dev, had_table, host, rand_signs, say

pytestmark = pytest.mark.gpu

FAST = [(172, 64), (28, 512), (28, 1024)]


@pytest.mark.parametrize("a,b", FAST)
@pytest.mark.parametrize("N", [1, 3, 6, 1027])
def test_pack_rotated_row_counts(a, b, N):
    if N > 1000 and a * b > 16384:
        N = 515  # more rows than workgroups that fit the chip at once
    say(f"pack_w4 rotated N={N} a={a} b={b}")
    check_w(workloads.weights(workloads.rng_for(N + a), N, a * b), a, b)


@pytest.mark.parametrize("a,b", FAST)
def test_pack_rotated_strided_and_misaligned_factor(a, b):
    """Rows with padding between them (NaN, never read), and a factor that is not 16-byte
    aligned."""
    say(f"pack_w4 strided rows, misaligned factor a={a} b={b}")
    K, N = a * b, 21
    w = workloads.weights(workloads.rng_for(a + 5), N, K)
    wide = torch.full((N, K + 24), float("nan"), dtype=torch.float16, device="cuda")
    wide[:, :K] = dev(w)
    ref = [host(t) for t in sq.pack_w4(dev(w), had_table(a), b)]
    got = [host(t) for t in sq.pack_w4(wide[:, :K], had_table(a), b)]
    for x, y in zip(got, ref):
        np.testing.assert_array_equal(x, y)
    flat = torch.empty(a * a + 1, dtype=torch.int8, device="cuda")
    h = flat[1:].view(a, a)
    h.copy_(had_table(a))
    gq, ga, gr = (host(t) for t in sq.pack_w4(dev(w), h, b))
    parity.assert_params_close(ga, ref[1])
    c, d = parity.unpack(gq, signed=True), parity.unpack(ref[0], signed=True)
    parity.code_flips(c, d)
    np.testing.assert_array_equal(gr, c.sum(1))


@pytest.mark.parametrize("a,b", FAST)
def test_pack_rotated_signs(a, b):
    """S H folded in: the codes of the sign-flipped weight rows, which is the same rotation."""
    say(f"pack_w4_ex signs a={a} b={b}")
    K, N = a * b, 9
    w = workloads.weights(workloads.rng_for(a + b), N, K)
    s = rand_signs(K, 7)
    got = [host(t) for t in sq.pack_w4(dev(w), had_table(a), b, signs=dev(s))]
    flipped = (w.astype(np.float32) * s.astype(np.float32)).astype(np.float16)
    ref = [host(t) for t in sq.pack_w4(dev(flipped), had_table(a), b)]
    for x, y in zip(got, ref):
        np.testing.assert_array_equal(x, y)


@pytest.mark.parametrize("a,b", FAST)
def test_pack_rotated_degenerate_rows(a, b):
    """Zero rows (alpha 1, codes 0), one impulse (every rotated value +-amax: codes +-7), the
    smallest fp16 subnormals, and the largest finite values."""
    say(f"pack_w4 degenerate rows a={a} b={b}")
    K = a * b
    w = np.zeros((5, K), dtype=np.float16)
    w[1, 3] = 0.5
    w[2, :] = np.float16(6e-8) * np.sign(ohad.dense_factor(a)[0].repeat(b)).astype(np.float16)
    w[3, :] = 65504.0
    w[4, ::7] = -0.01
    wq, wa, rs = (host(t) for t in sq.pack_w4(dev(w), had_table(a), b))
    c = parity.unpack(wq, signed=True)
    np.testing.assert_array_equal(rs, c.sum(1))
    assert wa[0] == 1.0 and not c[0].any()
    assert (np.abs(c[1]) == 7).all()
    op, owa, ors, oc = olin.pack_w4(w, ohad.dense_factor(a), b)
    parity.assert_params_close(wa, owa)
    parity.code_flips(c, oc)


@pytest.mark.parametrize("K", [8, 4096, 4104, 8192, 8200, 16384, 16392, 32768])
def test_pack_identity_row_lengths(K):
    """The register kernel's chunk counts: bit-exact (no rotation rounding)."""
    say(f"pack_w4 unrotated K={K}")
    w = workloads.weights(workloads.rng_for(K), 5, K)
    w[2] = 0
    w[3, :] = np.float16(6e-8)
    w[4, 0] = 65504.0
    assert check_w(w, 1, 1) == 0
