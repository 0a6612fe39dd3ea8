"""GPU: forward calls whose keys are split over several workgroups and merged (fewer queries than keys).

Sizes where the split can go wrong: a last split that is short or ends inside a tile, splits wholly or partly
beyond the diagonal of a query tile, one query, groups of heads, both head dimensions.  O and LSE are checked
against the fp64 oracle with the bounds of the unsplit forward, and nothing is written behind the scratch.
"""
import math

import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc
from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu

GUARD = 1024


@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,D,causal", [
    (1, 2, 1, 130, 1100, 64, True), (1, 4, 2, 1000, 1300, 128, True), (2, 3, 3, 1, 2000, 128, True), (1, 2, 2, 70, 1025, 64, False),
    (1, 8, 2, 257, 4100, 128, True), (1, 4, 1, 1023, 1024, 64, True), (1, 5, 5, 200, 1537, 128, False)])
def test_split_forward(B, Hq, Hkv, Nq, Nk, D, causal):
    g = torch.Generator().manual_seed(31 * Nq + Nk)
    q, k, v = (torch.randn(B, h, n, D, generator=g).to(torch.bfloat16) for h, n in ((Hq, Nq), (Hkv, Nk), (Hkv, Nk)))
    scale = 1 / math.sqrt(D)
    qd, kd, vd = q.cuda(), k.cuda(), v.cuda()
    o, lse = torch.full_like(qd, float("nan")), torch.full((B, Hq, Nq), float("nan"), device="cuda")
    n = attn.tk_attn_fwd_scratch_bytes(B, Hq, Hkv, Nq, Nk, D, causal)
    assert n > 0, "this shape is meant to be split"
    scratch = torch.full((n + GUARD,), 0xFF, dtype=torch.uint8, device="cuda")
    print(f"launch split B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} causal={causal}", flush=True)
    assert attn.tk_attn_fwd_rect_scratch(qd, kd, vd, o, lse, B, Hq, Hkv, Nq, Nk, D, causal, scale, scratch, n) == attn.TK_OK
    torch.cuda.synchronize()
    assert bool((scratch[n:] == 0xFF).all()), "wrote past the end of the scratch"
    o_ref, lse_ref = orc.rect_fwd(*(t.double().numpy() for t in (q, k, v)), causal, scale)
    err = np.abs(o.double().cpu().numpy() - o_ref)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
    assert np.abs(lse.double().cpu().numpy() - lse_ref).max() <= 1e-3
    # too little scratch, or none: the unsplit call, bit for bit
    o1, lse1, o2, lse2 = torch.empty_like(o), torch.empty_like(lse), torch.empty_like(o), torch.empty_like(lse)
    assert attn.tk_attn_fwd_rect(qd, kd, vd, o1, lse1, B, Hq, Hkv, Nq, Nk, D, causal, scale) == attn.TK_OK
    assert attn.tk_attn_fwd_rect_scratch(qd, kd, vd, o2, lse2, B, Hq, Hkv, Nq, Nk, D, causal, scale, scratch, n - 1) == attn.TK_OK
    assert torch.equal(o1, o2) and torch.equal(lse1, lse2)
    # the convenience function brings its own scratch, on another stream too
    o3, lse3 = attn.rect_fwd(qd, kd, vd, causal, scale)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    o4, lse4 = attn.rect_fwd(qd, kd, vd, causal, scale, stream=side)
    side.synchronize()
    torch.cuda.synchronize()
    for a, b in ((o, o3), (lse, lse3), (o, o4), (lse, lse4)):
        assert torch.equal(a, b)


def test_calls_that_are_not_split():
    for shape in ((1, 1, 1, 4096, 4096, 128, True), (1, 1, 1, 5000, 4096, 128, False), (1, 64, 64, 1024, 4096, 128, True),
                  (1, 2, 2, 100, 900, 64, True), (1, 2, 2, 4096, 100, 64, True), (1, 2, 2, 1, 4096, 96, False),
                  # two splits of few tiles and many rows: the merge would cost more than they save
                  (4, 16, 2, 322, 1529, 128, False), (1, 128, 32, 160, 1399, 64, False), (1, 163, 163, 86, 1380, 128, True)):
        assert attn.tk_attn_fwd_scratch_bytes(*shape) == 0, shape


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,causal", [(2, 4, 2, 130, 4100, False), (2, 2, 2, 200, 3000, True), (1, 8, 2, 1, 2500, False),
                                                   (2, 8, 2, 1, 9000, False), (40, 8, 4, 1, 4000, False)])
def test_masked_keys(B, Hq, Hkv, Nq, Nk, D, causal):
    """Keys that the caller masks with scores of -inf (one column of K holds the mask, the same column of Q ones): whole
    splits without a visible key add nothing.  One query: decode, on its own kernel and on the forward's."""
    g = torch.Generator().manual_seed(Nq + Nk + D)
    q, k, v = (torch.randn(B, h, n, D, generator=g).to(torch.bfloat16) for h, n in ((Hq, Nq), (Hkv, Nk), (Hkv, Nk)))
    q[..., D - 1] = 1.0
    k[..., D - 1] = 0.0
    for b in range(B):
        k[b, :, 300 + 77 * b:, D - 1] = float("-inf")        # the padding of a shorter sequence
    k[:, :, 70:200, D - 1] = float("-inf")                  # and whole tiles in between
    scale = 1 / math.sqrt(D)
    print(f"launch masked B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} causal={causal}", flush=True)
    if Nq == 1:
        o, lse = attn.decode(q.cuda(), k.cuda(), v.cuda(), scale)
    else:
        assert attn.tk_attn_fwd_scratch_bytes(B, Hq, Hkv, Nq, Nk, D, causal) > 0, "this shape is meant to be split"
        o, lse = attn.rect_fwd(q.cuda(), k.cuda(), v.cuda(), causal, scale)
    torch.cuda.synchronize()
    b = B - 1                                               # (the rows of one entry: the oracle walks every key in fp64)
    o_ref, lse_ref = orc.rect_fwd(*(t[b:b + 1].double().numpy() for t in (q, k, v)), causal, scale)
    assert np.isfinite(o_ref).all()
    for e in range(B):
        assert bool(torch.isfinite(o[e]).all()) and bool(torch.isfinite(lse[e]).all()), e
    err = np.abs(o[b:b + 1].double().cpu().numpy() - o_ref)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
    assert np.abs(lse[b:b + 1].double().cpu().numpy() - lse_ref).max() <= 1e-3
