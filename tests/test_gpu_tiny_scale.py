"""GPU: a scale so small that LSE / scale is no fp32 number; every key then has the weight 1 / N."""
import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D,B,H,N", [(64, 1, 2, 256), (128, 1, 2, 200), (128, 8, 16, 512)])
def test_smallest_scale(D, B, H, N):
    g = torch.Generator(device="cuda").manual_seed(D + N)
    q, k, v, d_o = (torch.randn(B, H, N, D, generator=g, device="cuda").to(torch.bfloat16) for _ in range(4))
    scale = 1e-38
    o, lse = torch.empty_like(q), torch.empty(B, H, N, device="cuda")
    dq, dk, dv = (torch.empty_like(q) for _ in range(3))
    size = attn.tk_attn_bwd_workspace_bytes(B, H, N, D)
    ws = torch.empty(size, dtype=torch.uint8, device="cuda")
    print(f"launch forward and backward B{B} H{H} N{N} D{D} scale {scale}", flush=True)
    assert attn.tk_attn_fwd(q, k, v, o, lse, B, H, N, D, False, scale) == attn.TK_OK
    assert attn.tk_attn_bwd_rect(q, k, v, o, d_o, lse, dq, dk, dv, B, H, H, N, N, D, False, scale, ws, size) == attn.TK_OK
    # P is rounded to bf16 (2^-9 of it), dV once more: 2^-8 of the sum of magnitudes bounds both
    mean = d_o.double().mean(2, keepdim=True).expand_as(dv)
    bound = 2.0**-8 * d_o.double().abs().mean(2, keepdim=True) + 1e-6
    assert ((dv.double() - mean).abs() <= bound).all()
    assert dq.float().abs().max() < 1e-30 and dk.float().abs().max() < 1e-30
