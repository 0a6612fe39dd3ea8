"""GPU: the dK/dV kernel with tiles of 256 keys, which large calls at D = 128 take.

It does the work of the kernel with 128-key tiles in the same order: every head of a large call has the bits of the same
head run alone, and so has dQ, which one form of the backward computes from the dS blocks that the kernel stores.  (That kernel is
checked against the oracle elsewhere.)  Lengths that end inside a tile, inside a wave's 64 keys and at either half of them.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn
from kernel_names import launched

pytestmark = pytest.mark.gpu

D = 128


def backward(q, k, v, d_o, causal, storing):
    B, Hq, Nq, _ = q.shape
    Hkv, Nk = k.shape[1:3]
    scale = 1 / math.sqrt(D)
    o, lse = torch.empty_like(q), torch.empty(B, Hq, Nq, device="cuda")
    assert attn.tk_attn_fwd_rect(q, k, v, o, lse, B, Hq, Hkv, Nq, Nk, D, causal, scale) == attn.TK_OK
    grads = tuple(torch.full_like(t, math.nan) for t in (q, k, v))
    size = attn.tk_attn_bwd_spill_workspace_bytes(B, Hq, Nq, Nk, D) if storing else attn.tk_attn_bwd_workspace_bytes(B, Hq, Nq, D)
    ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")
    assert attn.tk_attn_bwd_rect(q, k, v, o, d_o, lse, *grads, B, Hq, Hkv, Nq, Nk, D, causal, scale, ws, size) == attn.TK_OK
    return grads


@pytest.mark.parametrize("storing", [False, True])
@pytest.mark.parametrize("B,H,Nq,Nk,causal", [
    (8, 16, 512, 512, False), (8, 16, 1000, 420, False), (16, 16, 95, 200, False), (8, 8, 2048, 2048, True), (8, 8, 1300, 1300, True),
    (16, 8, 801, 801, True), (8, 8, 1135, 1300, True), (8, 8, 1236, 1300, True), (8, 8, 1665, 1665, True), (8, 8, 775, 3176, True)])
def test_heads_of_a_large_call(B, H, Nq, Nk, causal, storing):
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk)
    new = lambda n: torch.randn(B, H, n, D, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v, d_o = new(Nq), new(Nk), new(Nk), new(Nq)
    print(f"launch backward B{B} H{H} Nq{Nq} Nk{Nk} causal={causal} storing={storing}", flush=True)
    grads, names = launched(lambda: backward(q, k, v, d_o, causal, storing))
    assert any("attn_bwd_dkdv_wide_kernel" in n for n in names), names
    for b, h in {(0, 0), (B - 1, H - 1), (B // 2, 1)}:
        one, names = launched(lambda: backward(*(t[b:b + 1, h:h + 1].contiguous() for t in (q, k, v, d_o)), causal, storing))
        assert any("attn_bwd_dkdv_kernel" in n for n in names), names
        for name, x, y in zip(("dq", "dk", "dv"), grads, one):
            assert torch.equal(x[b, h], y[0, 0]), (name, b, h)


@pytest.mark.parametrize("B,Hq,Hkv,N,causal", [(8, 32, 16, 2048, True), (8, 48, 16, 500, False)])
def test_groups_of_a_large_call(B, Hq, Hkv, N, causal):
    """The stream of a key tile runs over the query heads of a group."""
    g = torch.Generator(device="cuda").manual_seed(N)
    new = lambda h: torch.randn(B, h, N, D, generator=g, device="cuda").to(torch.bfloat16)
    q, k, v, d_o = new(Hq), new(Hkv), new(Hkv), new(Hq)
    scale = 1 / math.sqrt(D)

    def dkdv(q, k, v, d_o):
        b, hq, hkv = q.shape[0], q.shape[1], k.shape[1]
        o, lse, delta = torch.empty_like(q), torch.empty(b, hq, N, device="cuda"), torch.empty(b, hq, N, device="cuda")
        assert attn.tk_attn_fwd_gqa(q, k, v, o, lse, b, hq, hkv, N, D, causal, scale) == attn.TK_OK
        assert attn.tk_attn_bwd_delta(o, d_o, delta, b, hq, N, D) == attn.TK_OK
        dk, dv = torch.full_like(k, math.nan), torch.full_like(v, math.nan)
        assert attn.tk_attn_bwd_dkdv_gqa(q, k, v, d_o, lse, delta, dk, dv, b, hq, hkv, N, D, causal, scale) == attn.TK_OK
        return dk, dv

    print(f"launch dK/dV B{B} Hq{Hq} Hkv{Hkv} N{N} causal={causal}", flush=True)
    all_heads, names = launched(lambda: dkdv(q, k, v, d_o))
    assert any("attn_bwd_dkdv_wide_kernel" in n for n in names), names
    group = Hq // Hkv
    for b, h in ((0, 0), (B - 1, Hkv - 1)):
        heads = slice(h * group, (h + 1) * group)
        one, names = launched(lambda: dkdv(q[b:b + 1, heads].contiguous(), k[b:b + 1, h:h + 1].contiguous(), v[b:b + 1, h:h + 1].contiguous(), d_o[b:b + 1, heads].contiguous()))
        assert any("attn_bwd_dkdv_kernel" in n for n in names), names
        for name, x, y in zip(("dk", "dv"), all_heads, one):
            assert torch.equal(x[b, h], y[0, 0]), (name, b, h)
