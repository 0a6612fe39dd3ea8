"""GPU: backward with the smallest scales and scores that are large all the same: Q and K as large as the scale is small.

The scores differ by a few units.  Checked in fp64 for one head, by the norm of the difference: 1e-2, four times what the roundings
to bf16 of P, dS and O leave in the gradients.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storing", [False, True])
@pytest.mark.parametrize("scale", [2e-38, 5e-37, 2e-36, 3e-30])
@pytest.mark.parametrize("D,B,H,N,causal", [(64, 1, 2, 256, False), (64, 1, 2, 333, True), (128, 1, 2, 200, False), (128, 1, 2, 384, True), (128, 8, 16, 512, False), (128, 8, 8, 1300, True)])
def test_small_scale(D, B, H, N, causal, scale, storing):
    g = torch.Generator(device="cuda").manual_seed(D + N)
    q, k, v, d_o = (torch.randn(B, H, N, D, generator=g, device="cuda") for _ in range(4))
    large = math.sqrt(1 / (scale * math.sqrt(D)))                  # (scores of the ordinary size)
    q, k, v, d_o = (t.to(torch.bfloat16) for t in (q * large, k * large, v, d_o))
    o, lse = torch.empty_like(q), torch.empty(B, H, N, device="cuda")
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    size = attn.tk_attn_bwd_spill_workspace_bytes(B, H, N, N, D) if storing else attn.tk_attn_bwd_workspace_bytes(B, H, N, D)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    print(f"launch forward and backward B{B} H{H} N{N} D{D} causal={causal} scale {scale} storing={storing}", flush=True)
    assert attn.tk_attn_fwd(q, k, v, o, lse, B, H, N, D, causal, scale) == attn.TK_OK
    assert attn.tk_attn_bwd_rect(q, k, v, o, d_o, lse, dq, dk, dv, B, H, H, N, N, D, causal, scale, ws, size) == attn.TK_OK
    qd, kd, vd, gd = (t[0, 0].double() for t in (q, k, v, d_o))
    s = qd @ kd.T * scale
    if causal:
        s = s.masked_fill(torch.ones(N, N, dtype=torch.bool, device="cuda").triu(1), -math.inf)
    p = torch.softmax(s, -1)
    ds = p * (gd @ vd.T - ((p @ vd) * gd).sum(-1, keepdim=True))
    for name, x, ref in (("o", o, p @ vd), ("dv", dv, p.T @ gd), ("dk", dk, scale * ds.T @ qd), ("dq", dq, scale * ds @ kd)):
        err = (x[0, 0].double() - ref).norm() / ref.norm()
        assert err <= 1e-2, (name, float(err))
