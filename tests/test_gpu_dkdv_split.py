"""GPU: backward calls whose queries are split over several workgroups of the dK/dV kernel.

The query heads of a group, the queries of a head (cross-attention) and both.  Odd and even tile counts, a length inside
the last key tile, parts of unequal length, groups that split fully or in part, more than 16 causal key tiles (a workgroup
then takes two, one pass behind the other), both forms of the backward.  Against the fp64 oracle, and with nothing written
behind the buffers.
"""
import math

import pytest
import torch

from grad_check import check_grad
from oracle import attn_oracle as orc
from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu

GUARD = 1024


@pytest.mark.parametrize("spill", [False, True], ids=["recompute", "spill"])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,D,causal", [
    (1, 4, 1, 256, 256, 128, True), (2, 8, 2, 333, 333, 128, True), (1, 6, 2, 300, 1000, 64, True), (1, 8, 1, 700, 130, 128, False),
    (1, 8, 1, 513, 513, 64, True), (5, 12, 2, 257, 1500, 64, False),
    (1, 4, 1, 2200, 2200, 128, True), (1, 8, 2, 2100, 2100, 64, True), (2, 4, 2, 300, 2500, 64, True), (1, 6, 1, 400, 2177, 128, True),
    (2, 4, 4, 1100, 300, 64, False), (1, 2, 2, 4000, 70, 64, False), (1, 3, 3, 2049, 129, 128, False), (1, 6, 3, 1090, 600, 128, False)])
def test_split_backward(B, Hq, Hkv, Nq, Nk, D, causal, spill):
    g = torch.Generator().manual_seed(17 * Nq + Nk + D)
    q, k, v, d_o = (torch.randn(B, h, n, D, generator=g).to(torch.bfloat16) for h, n in ((Hq, Nq), (Hkv, Nk), (Hkv, Nk), (Hq, Nq)))
    scale = 1 / math.sqrt(D)
    qd, kd, vd, dod = (t.cuda() for t in (q, k, v, d_o))
    o, lse = attn.rect_fwd(qd, kd, vd, causal, scale)
    n_ws = (attn.tk_attn_bwd_spill_workspace_bytes(B, Hq, Nq, Nk, D) if spill else attn.tk_attn_bwd_workspace_bytes(B, Hq, Nq, D))
    n = attn.tk_attn_bwd_scratch_bytes(B, Hq, Hkv, Nq, Nk, D, causal, n_ws)
    # (the storing form needs scratch only where the queries of a head are split: its workspace has room for the rest)
    assert (spill and (causal or n == 0)) or n >= 2 * 8 * B * Hkv * Nk * D, "this shape is meant to be split"
    ws = torch.full((n_ws + GUARD,), 0xFF, dtype=torch.uint8, device="cuda")
    scratch = torch.full((n + GUARD,), 0xFF, dtype=torch.uint8, device="cuda")
    dq, dk, dv = torch.full_like(qd, float("nan")), torch.full_like(kd, float("nan")), torch.full_like(vd, float("nan"))
    print(f"launch split backward B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} D{D} causal={causal} spill={spill}", flush=True)
    assert attn.tk_attn_bwd_rect_scratch(qd, kd, vd, o, dod, lse, dq, dk, dv, B, Hq, Hkv, Nq, Nk, D, causal, scale,
                                         ws, n_ws, scratch, n) == attn.TK_OK
    torch.cuda.synchronize()
    assert bool((ws[n_ws:] == 0xFF).all()) and bool((scratch[n:] == 0xFF).all()), "wrote past the end of a buffer"
    refs = orc.rect_bwd(*(t.double().numpy() for t in (q, k, v, d_o)), causal, scale)
    for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
        check_grad(got.double().cpu().numpy(), ref, name)
    # the convenience function takes the same way, on another stream too
    again = attn.rect_bwd(qd, kd, vd, o, dod, lse, causal, scale, ws[:n_ws])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    other = attn.rect_bwd(qd, kd, vd, o, dod, lse, causal, scale, ws[:n_ws], stream=side)
    side.synchronize()
    torch.cuda.synchronize()
    for a, b, c in zip((dq, dk, dv), again, other):
        assert torch.equal(a, b) and torch.equal(a, c)
    # a workspace with room for dS but not for partial sums, or no scratch: unsplit, and as good
    room = 8 * B * Hq * Nk * D if spill else 0
    for t in (dq, dk, dv):
        t.fill_(float("nan"))
    assert attn.tk_attn_bwd_rect(qd, kd, vd, o, dod, lse, dq, dk, dv, B, Hq, Hkv, Nq, Nk, D, causal, scale, ws, n_ws - room) == attn.TK_OK
    for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), refs):
        check_grad(got.double().cpu().numpy(), ref, name)


def test_calls_that_are_not_split():
    # where the partial sums cost more than the shorter streams save: few blocks, and pairs as long as the single tiles were
    for shape in ((5, 32, 16, 268, 268, 64, False), (3, 32, 8, 309, 1060, 128, True), (8, 32, 16, 369, 369, 64, True), (1, 8, 8, 1000, 1000, 64, True),
                  (1, 8, 2, 255, 255, 128, True), (16, 32, 8, 4096, 4096, 128, True)):
        n = attn.tk_attn_bwd_workspace_bytes(shape[0], shape[1], shape[3], shape[5])
        assert attn.tk_attn_bwd_scratch_bytes(*shape, n) == 0, shape
    for shape in ((2, 16, 4, 1001, 1001, 128, True), (1, 32, 8, 2048, 2048, 64, True), (1, 4, 4, 4096, 64, 64, False)):
        n = attn.tk_attn_bwd_workspace_bytes(shape[0], shape[1], shape[3], shape[5])
        assert attn.tk_attn_bwd_scratch_bytes(*shape, n) > 0, shape
