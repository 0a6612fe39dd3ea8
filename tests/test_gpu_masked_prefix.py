"""GPU: keys that the caller masks with scores of -inf, ahead of the visible ones (a left-padded batch) and a tile here and there.

One column of K holds the mask, the same column of Q ones.  O is checked in fp64 to within the two roundings to bf16, of P and of O:
2^-8 * (sum_j P_j |V_j| + |O|), and 1e-4 for all that happens in fp32.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


def masked_inputs(B, Hq, Hkv, Nq, Nk, D, padding):
    """padding: keys masked at the front, or "holes": every second tile of 64 keys, the first one of any split among them"""
    g = torch.Generator(device="cuda").manual_seed(Nq + Nk + D)
    q, k, v = (torch.randn(B, h, n, D, generator=g, device="cuda").to(torch.bfloat16) for h, n in ((Hq, Nq), (Hkv, Nk), (Hkv, Nk)))
    q[..., D - 1] = 1.0
    mask = torch.zeros(Nk, device="cuda")
    if padding == "holes":
        mask[(torch.arange(Nk, device="cuda") // 64) % 2 == 0] = -math.inf
    else:
        mask[:padding] = -math.inf
    k[..., D - 1] = mask.to(torch.bfloat16)
    return q, k, v


def check(o, lse, q, k, v, causal, scale):
    B, Hq, Nq, _ = q.shape
    Hkv, Nk = k.shape[1:3]
    assert bool(torch.isfinite(o).all()) and bool(torch.isfinite(lse).all())
    for b, h in {(0, 0), (B - 1, Hq - 1), (B // 2, Hq // 3)}:
        kv = h // (Hq // Hkv)
        s = q[b, h].double() @ k[b, kv].double().T * scale
        if causal:
            i = torch.arange(Nq, device="cuda")[:, None] + (Nk - Nq)
            s = s.masked_fill(torch.arange(Nk, device="cuda")[None, :] > i, -math.inf)
        p, vd = torch.softmax(s, -1), v[b, kv].double()
        o_ref = p @ vd
        err = (o[b, h].double() - o_ref).abs() / ((p @ vd.abs() + o_ref.abs()) / 256 + 1e-4)
        assert err.max() <= 1, (b, h, err.max())
        assert (lse[b, h].double() - torch.logsumexp(s, -1)).abs().max() <= 1e-3, (b, h)


@pytest.mark.parametrize("padding", [64, 128, 700, "holes"])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,D,causal", [
    (2, 4, 2, 130, 4100, 64, False), (2, 4, 2, 130, 4100, 128, False), (2, 2, 2, 200, 3000, 64, True), (2, 2, 2, 200, 3000, 128, True),
    (1, 2, 2, 33, 2500, 64, False), (4, 8, 4, 512, 4096, 64, True), (4, 8, 4, 512, 4096, 128, True), (3, 8, 8, 500, 8192, 128, False)])
def test_split_calls(B, Hq, Hkv, Nq, Nk, D, causal, padding):
    q, k, v = masked_inputs(B, Hq, Hkv, Nq, Nk, D, padding)
    assert attn.tk_attn_fwd_scratch_bytes(B, Hq, Hkv, Nq, Nk, D, causal) > 0, "this shape is meant to be split"
    print(f"launch masked split B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} causal={causal} {padding}", flush=True)
    o, lse = attn.rect_fwd(q, k, v, causal, 1 / math.sqrt(D))
    check(o, lse, q, k, v, causal, 1 / math.sqrt(D))


@pytest.mark.parametrize("padding", [64, 128, 700, "holes"])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,D,causal", [
    (2, 16, 2, 900, 3000, 64, False), (2, 16, 2, 900, 3000, 64, True), (2, 16, 2, 1200, 3000, 128, False), (2, 16, 2, 1200, 3000, 128, True),
    (16, 16, 16, 40, 1000, 64, False), (16, 16, 16, 40, 1000, 128, False), (4, 16, 16, 1024, 1024, 128, False), (1, 2, 2, 300, 900, 64, False),
    (1, 4, 4, 100, 128, 64, False)])
def test_unsplit_calls(B, Hq, Hkv, Nq, Nk, D, causal, padding):
    """Whether a call is split depends on its sizes; what it answers does not."""
    if padding != "holes" and padding >= Nk:
        padding = Nk - 1
    q, k, v = masked_inputs(B, Hq, Hkv, Nq, Nk, D, padding)
    assert attn.tk_attn_fwd_scratch_bytes(B, Hq, Hkv, Nq, Nk, D, causal) == 0, "this shape is not meant to be split"
    print(f"launch masked B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} causal={causal} {padding}", flush=True)
    o, lse = attn.rect_fwd(q, k, v, causal, 1 / math.sqrt(D))
    check(o, lse, q, k, v, causal, 1 / math.sqrt(D))


@pytest.mark.parametrize("padding", [64, 700, "holes"])
@pytest.mark.parametrize("Hq,D", [(96, 64), (96, 128), (8, 128)])
def test_decode(Hq, D, padding):
    """More than 64 heads on a key/value head: the rows of a tile of the forward kernel."""
    q, k, v = masked_inputs(2, Hq, 1, 1, 6000, D, padding)
    print(f"launch masked decode Hq{Hq} D{D} {padding}", flush=True)
    o, lse = attn.decode(q, k, v, 1 / math.sqrt(D))
    check(o, lse, q, k, v, False, 1 / math.sqrt(D))
