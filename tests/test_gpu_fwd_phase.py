"""GPU: the forward kernel in phases, with one group of waves and with two.

Both forms do the same arithmetic, so a head of a call that is large enough for two groups (256-row tiles) has the bits
of the same head run alone (one group).  The scores either stay within one range or grow along the keys, so that later
tiles have to be done again against their own maximum.  Sampled heads are checked in fp64, each element of O to within the
two roundings to bf16, of P and of O, each at most 2^-8 of the value: 2^-8 * (sum_j P_j |V_j| + |O|); and 1e-4 for all
that happens in fp32.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


def reference(q, k, v, causal, scale):
    s = q.double() @ k.double().T * scale
    if causal:
        i = torch.arange(q.shape[0], device=q.device)[:, None] + (k.shape[0] - q.shape[0])
        s = s.masked_fill(torch.arange(k.shape[0], device=q.device)[None, :] > i, -math.inf)
    p = torch.softmax(s, -1)
    return p @ v.double(), p @ v.double().abs(), torch.logsumexp(s, -1)


@pytest.mark.parametrize("growing", [False, True])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,D,causal", [
    (4, 16, 16, 1024, 1024, 128, False), (4, 16, 4, 993, 993, 128, False), (2, 16, 16, 4096, 4096, 128, True),
    (2, 16, 16, 4001, 4001, 128, True), (2, 32, 8, 1000, 3900, 128, False),      # two groups
    (1, 3, 3, 129, 129, 128, True), (2, 2, 1, 64, 64, 128, False), (1, 4, 4, 200, 1000, 64, True), (1, 2, 2, 1217, 1217, 64, True),
    (3, 4, 4, 256, 192, 64, False), (1, 5, 5, 1, 129, 64, True)])
def test_forward_phases(B, Hq, Hkv, Nq, Nk, D, causal, growing):
    g = torch.Generator(device="cuda").manual_seed(Nq + 3 * Nk)
    new = lambda h, n: torch.randn(B, h, n, D, generator=g, device="cuda")
    q, k, v = new(Hq, Nq), new(Hkv, Nk), new(Hkv, Nk)
    if growing:
        k *= torch.linspace(0.1, 30, Nk, device="cuda")[:, None]
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    scale = 1 / math.sqrt(D)
    print(f"launch forward B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} causal={causal} growing={growing}", flush=True)
    o, lse = torch.full_like(q, math.nan), torch.full((B, Hq, Nq), math.nan, device="cuda")
    assert attn.tk_attn_fwd_rect(q, k, v, o, lse, B, Hq, Hkv, Nq, Nk, D, causal, scale) == attn.TK_OK
    for b, h in {(0, 0), (B - 1, Hq - 1), (B // 2, Hq // 3)}:
        kv = h // (Hq // Hkv)
        one = q[b:b + 1, h:h + 1].contiguous(), k[b:b + 1, kv:kv + 1].contiguous(), v[b:b + 1, kv:kv + 1].contiguous()
        o1, l1 = torch.empty_like(one[0]), torch.empty(1, 1, Nq, device="cuda")
        assert attn.tk_attn_fwd_rect(*one, o1, l1, 1, 1, 1, Nq, Nk, D, causal, scale) == attn.TK_OK
        assert torch.equal(o[b, h], o1[0, 0]) and torch.equal(lse[b, h], l1[0, 0]), (b, h)
        o_ref, o_abs, lse_ref = reference(one[0][0, 0], one[1][0, 0], one[2][0, 0], causal, scale)
        err = (o[b, h].double() - o_ref).abs() / ((o_abs + o_ref.abs()) / 256 + 1e-4)
        assert err.max() <= 1, err.max()
        assert (lse[b, h].double() - lse_ref).abs().max() <= 1e-3
