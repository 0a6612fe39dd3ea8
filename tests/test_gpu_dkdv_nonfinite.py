"""GPU: infinities and NaN in the backward's inputs do not get further with 256-key tiles than with 128-key tiles.

A head of a large call against the same head alone, which takes the 128-key kernel: wherever that has a number or an infinity,
the large call has the same one.  (Masked blocks of the 128-key tiles multiply 0 by what the mask hides and may be NaN; the
256-key tiles leave out more of those.)  Under the causal mask the rows hit lie in the first half of a 256-key tile: none of them
sees a key of the second half.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn
from kernel_names import launched

pytestmark = pytest.mark.gpu

D = 128


def backward(q, k, v, d_o, lse, delta, causal, storing):
    B, Hq, N, _ = q.shape
    Hkv = k.shape[1]
    dk, dv = torch.empty_like(k), torch.empty_like(v)
    if storing:
        ds = torch.empty(attn.tk_attn_bwd_ds_bytes(B, Hq, N, N, D), dtype=torch.uint8, device="cuda")
        assert attn.tk_attn_bwd_dkdv_ds(q, k, v, d_o, lse, delta, dk, dv, ds, B, Hq, Hkv, N, D, causal, 1 / math.sqrt(D)) == attn.TK_OK
    else:
        assert attn.tk_attn_bwd_dkdv_gqa(q, k, v, d_o, lse, delta, dk, dv, B, Hq, Hkv, N, D, causal, 1 / math.sqrt(D)) == attn.TK_OK
    return dk, dv


@pytest.mark.parametrize("what", ["dO inf", "dO nan", "Q nan", "LSE nan"])
@pytest.mark.parametrize("B,Hq,Hkv,N,causal,storing", [
    (8, 16, 16, 512, False, False), (8, 16, 16, 512, False, True), (8, 16, 16, 500, False, False), (8, 16, 16, 500, False, True),
    (8, 8, 8, 2048, True, False), (8, 8, 8, 2048, True, True), (8, 16, 16, 1665, True, False), (8, 16, 16, 1665, True, True),
    (8, 32, 16, 2048, True, False)])        # (a group alone and storing dS is split, and sums in another order)
def test_nonfinite(B, Hq, Hkv, N, causal, storing, what):
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k, v, d_o = (torch.randn(B, h, N, D, generator=g, device="cuda").to(torch.bfloat16) for h in (Hq, Hkv, Hkv, Hq))
    lse, delta = torch.full((B, Hq, N), math.log(N) + 0.5, device="cuda"), torch.randn(B, Hq, N, generator=g, device="cuda")
    rows = [3, 300, 380]
    if what == "dO inf":
        d_o[:, :, rows, 5] = math.inf
    elif what == "dO nan":
        d_o[:, :, rows] = math.nan
    elif what == "Q nan":
        q[:, :, rows] = math.nan
    else:
        lse[:, :, rows] = math.nan
    print(f"launch dK/dV B{B} Hq{Hq} Hkv{Hkv} N{N} causal={causal} storing={storing} {what}", flush=True)
    large, names = launched(lambda: backward(q, k, v, d_o, lse, delta, causal, storing))
    assert any("attn_bwd_dkdv_wide_kernel" in n for n in names), names
    group = Hq // Hkv
    for b, h in ((0, 0), (B - 1, Hkv - 1)):
        heads = slice(h * group, (h + 1) * group)
        one = [t[b:b + 1, heads].clone() for t in (q, d_o, lse, delta)]
        kv = [t[b:b + 1, h:h + 1].clone() for t in (k, v)]
        alone, names = launched(lambda: backward(one[0], *kv, *one[1:], causal, storing))
        assert any("attn_bwd_dkdv_kernel" in n for n in names), names
        for name, x, y in zip(("dk", "dv"), large, alone):
            kept = ~y[0, 0].isnan()
            assert bool(kept.any()) or not causal or N <= 512, name
            assert torch.equal(x[b, h][kept], y[0, 0][kept]), (name, b, h)
