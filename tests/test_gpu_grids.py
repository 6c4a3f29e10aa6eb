"""Calls of more workgroups than one grid holds (2^32 threads), at the smallest sizes that need
them: the results around every part's ends are those of calls on those rows alone."""

import pytest
import torch

from paper_2405_16406_amd import sq

from test_gpu_parity import say

pytestmark = pytest.mark.gpu


def pieces(n):
    """Rows around the ends of parts of 2^23 - 1 and 2^24 - 1 rows, and of the call."""
    cuts = [0, (1 << 22) - 1, 1 << 23, 2 * ((1 << 23) - 1), 1 << 24, n]
    return [slice(max(0, c - 4), min(n, c + 4)) for c in cuts if c <= n]


@pytest.mark.parametrize("bits,group", [(4, 8), (8, 8), (4, 4)])
def test_quantize_many_rows(bits, group):
    M, K = (1 << 24) + 3, 8
    say(f"had_quant_act M={M} K={K} bits={bits} group={group}")
    x = torch.randn((M, K), dtype=torch.float16, device="cuda")
    got = sq.had_quant_act(x, bits=bits, group=group, dbg=True)
    for s in pieces(M):
        for u, v in zip(got, sq.had_quant_act(x[s], bits=bits, group=group, dbg=True)):
            assert torch.equal(u[s], v), s


@pytest.mark.parametrize("pow2", [1, 8])
def test_pack_many_rows(pow2):
    N, K = (1 << 24) + 3, 8
    say(f"pack_w4 N={N} K={K} rotation {pow2}")
    w = torch.randn((N, K), dtype=torch.float16, device="cuda")
    got = sq.pack_w4(w, None, pow2)
    for s in pieces(N):
        for u, v in zip(got, sq.pack_w4(w[s], None, pow2)):
            assert torch.equal(u[s], v), s


@pytest.mark.parametrize("param", [torch.float32, torch.float16])
@pytest.mark.parametrize("split", [False, True])
def test_attention_many_heads(split, param):
    B = (1 << 23) + 3
    say(f"attention B={B} S=1 H=1 split={split} {param}")
    q = torch.randn((B, 1, 128), dtype=torch.float16, device="cuda")
    cache = []
    for _ in range(2):
        cache += [torch.randint(0, 256, (B, 1, 1, 64), dtype=torch.uint8, device="cuda")]
        cache += [torch.rand((B, 1, 1, 1), device="cuda").to(param) for _ in range(2)]
    attn = sq.attn_decode_kv4_split_noalloc if split else sq.attn_decode_kv4
    got = attn(q, *cache, out=torch.full_like(q, float("nan")))
    for s in pieces(B):
        assert torch.equal(got[s], attn(q[s], *(c[s] for c in cache), out=torch.empty_like(q[s]))), s
