"""Rotation of activation rows on the one-row kernel and, for many rows of H_172 (x) S_64, the
row-pair kernel: the line between the two, every code form, and views at any alignment."""

import numpy as np
import pytest
import torch

from oracle import hadamard as ohad
from paper_2405_16406_amd import sq, workloads

import parity
from test_gpu_parity import check_act_var, dev, had_table, host, rand_signs, say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("var", [False, True])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("a,b", [(172, 64), (28, 512), (28, 1024)])
def test_row_results_do_not_depend_on_row_count(a, b, bits, var):
    """Both kernels take the same fp32 steps per row, so a row's results are the same bytes
    alone, at the last row count of the one-row kernel and at the first of the other."""
    K = a * b
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    M = 3 * cus + 1
    say(f"had_quant_act a={a} b={b} bits={bits} var={var}: rows 1, {M - 1}, {M}")
    x = workloads.outlier_acts(workloads.rng_for(a + b + bits), M, K, K // 100, 50.0)
    kw = dict(bits=bits, clip=0.9, signs=dev(rand_signs(K, 3))) if var else dict(bits=bits)
    full = [host(t) for t in sq.had_quant_act(dev(x), had_table(a), b, **kw)[:3]]
    for rows in (slice(0, M - 1), slice(0, 1), slice(M - 1, M)):
        part = [host(t) for t in sq.had_quant_act(dev(x[rows]), had_table(a), b, **kw)[:3]]
        for u, v in zip(part, full):
            np.testing.assert_array_equal(u, v[rows])


@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("a,b,M", [(172, 64, 5), (172, 64, 1025), (28, 512, 5), (28, 1024, 5)])
def test_factor_and_signs_at_odd_addresses(a, b, M, bits):
    say(f"had_quant_act_ex a={a} b={b} M={M} bits={bits}: H_a at +1 byte, signs at +3")
    K = a * b
    x = workloads.outlier_acts(workloads.rng_for(a + M), M, K, K // 100, 50.0)
    s = rand_signs(K, 11)
    hbuf = torch.empty(a * a + 16, dtype=torch.int8, device="cuda")[1:1 + a * a].view(a, a)
    hbuf.copy_(had_table(a))
    sbuf = torch.empty(K + 16, dtype=torch.int8, device="cuda")[3:3 + K]
    sbuf.copy_(dev(s.astype(np.int8)))
    rows = np.array([0, M // 2, M - 1])
    check_act_var(x, a, b, bits=bits, clip=0.95, signs=s, h_gpu=hbuf, s_gpu=sbuf, sample_rows=rows)


def near_constant(a, b, s):
    """Rows whose rotated values are 2^15 plus a few steps e = 2^-8 .. 2^11, all exact in fp32: an
    impulse against a factor whose first row is ones, and three or five entries +-e.  Returns x
    (its signs flipped by s), the factor, and the unscaled rotated rows."""
    rng = workloads.rng_for(a + b)
    h = ohad.dense_factor(a).astype(np.int64)
    h *= h[0]  # columns flipped: still a Hadamard matrix
    syl = ohad.sylvester(b).astype(np.int64)
    xs, ys = [], []
    for k in (-8, -7, -5, -2, 1, 4, 6, 8, 11):
        for m in (3, 5):
            e = 2.0 ** k
            x, y = np.zeros((a, b)), np.full((a, b), 2.0 ** 15)
            x[0, 0] = 2.0 ** 15
            for i in rng.choice(np.arange(1, a * b), m, replace=False):
                v = e * rng.choice([-1, 1])
                x[i // b, i % b] = v
                y += v * np.outer(h[i // b], syl[i % b])
            assert y.max() - y.min() == 2 * m * e, "every sign pattern of the entries occurs"
            xs.append(x.ravel() * s)
            ys.append(y.ravel())
    return np.array(xs).astype(np.float16), h.astype(np.int8), np.array(ys, dtype=np.float32)


@pytest.mark.parametrize("signs", [False, True])
@pytest.mark.parametrize("bits", [4, 8])
@pytest.mark.parametrize("a,b,M", [(172, 64, 18), (172, 64, 1100), (28, 512, 18), (28, 1024, 18)])
def test_near_constant_rows(a, b, M, bits, signs):
    """A row's range down to 2^-22 of its values: eq. 1's steps on the exact rotated values give
    whole code arguments (multiples of L / 3 or L / 5), so the codes are equal bit for bit."""
    say(f"had_quant_act near-constant rows a={a} b={b} M={M} bits={bits} signs={signs}")
    K, L = a * b, np.float32(2 ** bits - 1)
    s = rand_signs(K, 5) if signs else np.ones(K)
    x, h, y = (np.resize(t, (M, K)) if t.shape[-1] == K else t for t in near_constant(a, b, s))
    q, al, be, rot = sq.had_quant_act(dev(x), dev(h), b, bits=bits, dbg=True, signs=dev(s.astype(np.int8)) if signs else None)
    s_n = np.float32(1.0 / np.sqrt(float(K)))
    np.testing.assert_array_equal(host(rot), y * s_n)
    mn, mx = y.min(1, keepdims=True), y.max(1, keepdims=True)
    alpha = (mx - mn) / L
    codes = np.rint((y - mn) * (np.float32(1) / alpha)).astype(np.int64)
    got = host(q).astype(np.int64) if bits == 8 else parity.unpack(host(q), signed=False)
    np.testing.assert_array_equal(got, codes)
    np.testing.assert_array_equal(host(al), alpha * s_n)
    np.testing.assert_array_equal(host(be), mn * s_n)
