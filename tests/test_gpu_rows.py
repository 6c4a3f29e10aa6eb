"""Rotation of activation rows on the one-row kernel and, for many rows of H_172 (x) S_64, the
row-pair kernel: the line between the two, every code form, and views at any alignment."""

import numpy as np
import pytest
import torch

from paper_2405_16406_amd import sq, workloads

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
