"""GPU: values near the end of the number range, where O is accumulated before the division by the sum.

The first tile of keys scores 0, the later ones x in the base-2 exponent, so that a sum taken against the first maximum is
up to 2^x too large.  64 exponentials of at most 2^8 each are 2^14 a tile; V is as large as leaves Nk / 64 times that finite.
O is checked in fp64 to within the two roundings to bf16, of P and of O, and 1e-4 of the largest V for what happens in fp32.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("x", [2.0, 7.0, 10.8])
@pytest.mark.parametrize("B,H,Nq,Nk,D,causal", [
    (1, 2, 1024, 1024, 64, False), (1, 2, 1500, 1500, 64, True), (1, 2, 1024, 1024, 128, True), (4, 16, 1024, 1024, 128, False), (2, 16, 3000, 3000, 128, True),
    (1, 2, 130, 3900, 64, False), (1, 2, 130, 3900, 128, True), (3, 8, 500, 3900, 128, True)])
def test_large_values(B, H, Nq, Nk, D, causal, x):
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk + D)
    q, k, v = (torch.randn(B, H, n, D, generator=g, device="cuda") for n in (Nq, Nk, Nk))
    scale = 1 / math.sqrt(D)
    q *= 0.1
    q[..., 0] = 1.0
    k[..., 0] = 0.0
    k[:, :, 64:, 0] = x * math.log(2) / scale
    largest = 3e38 / (2**14 * Nk / 64)
    v = (0.75 + 0.05 * v.clamp(-5, 5)) * largest        # (of one sign: the sums do not cancel)
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    print(f"launch forward B{B} H{H} Nq{Nq} Nk{Nk} D{D} causal={causal} x={x}", flush=True)
    o, lse = attn.rect_fwd(q, k, v, causal, scale)
    assert bool(torch.isfinite(o).all()) and bool(torch.isfinite(lse).all())
    for b, h in {(0, 0), (B - 1, H - 1)}:
        s = q[b, h].double() @ k[b, h].double().T * scale
        if causal:
            i = torch.arange(Nq, device="cuda")[:, None] + (Nk - Nq)
            s = s.masked_fill(torch.arange(Nk, device="cuda")[None, :] > i, -math.inf)
        p, vd = torch.softmax(s, -1), v[b, h].double()
        o_ref = p @ vd
        err = (o[b, h].double() - o_ref).abs() / ((p @ vd.abs() + o_ref.abs()) / 256 + 1e-4 * largest)
        assert err.max() <= 1, (b, h, err.max())
        assert (lse[b, h].double() - torch.logsumexp(s, -1)).abs().max() <= 1e-3, (b, h)


@pytest.mark.parametrize("step", [5.0, 40.0])
@pytest.mark.parametrize("B,H,Nq,Nk,D,causal", [(1, 2, 1024, 1024, 64, False), (4, 16, 1024, 1024, 128, False), (1, 2, 130, 3900, 128, True), (1, 2, 33, 700, 64, True)])
def test_small_values(B, H, Nq, Nk, D, causal, step):
    """Scores that grow by 2^step from tile to tile, so that tiles are done again with room above them, and the smallest V."""
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk + D)
    q, k, v = (torch.randn(B, H, n, D, generator=g, device="cuda") for n in (Nq, Nk, Nk))
    scale = 1 / math.sqrt(D)
    q[..., 0] = 1.0
    k[..., 0] = (torch.arange(Nk, device="cuda") // 64) * (step * math.log(2) / scale)
    q, k, v = q.to(torch.bfloat16), k.to(torch.bfloat16), (v * 1e-36).to(torch.bfloat16)
    print(f"launch forward B{B} H{H} Nq{Nq} Nk{Nk} D{D} causal={causal} step={step}", flush=True)
    o, lse = attn.rect_fwd(q, k, v, causal, scale)
    for b, h in {(0, 0), (B - 1, H - 1)}:
        s = q[b, h].double() @ k[b, h].double().T * scale
        if causal:
            i = torch.arange(Nq, device="cuda")[:, None] + (Nk - Nq)
            s = s.masked_fill(torch.arange(Nk, device="cuda")[None, :] > i, -math.inf)
        p, vd = torch.softmax(s, -1), v[b, h].double()
        o_ref = p @ vd
        # an fp32 number of 1e-36 / 2^16 has 12 bits of its own left, 2^-13 of it is lost in each addition's rounding
        err = (o[b, h].double() - o_ref).abs() / ((p @ vd.abs() + o_ref.abs()) / 256 + 1e-3 * 1e-36)
        assert err.max() <= 1, (b, h, err.max())
        assert (lse[b, h].double() - torch.logsumexp(s, -1)).abs().max() <= 1e-3 + 1e-6 * lse[b, h].abs().max(), (b, h)
