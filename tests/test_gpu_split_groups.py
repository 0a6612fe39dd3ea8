"""GPU: split forward calls with workgroups of 256 query rows (D = 128): lengths that end inside a tile and inside a wave, splits that
lie wholly beyond the diagonal of a query tile, groups of heads, keys that the caller masks.  Checked in fp64 as the other split calls.
And calls of few rows at D = 64 that are not split but take another kernel with scratch.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn
from kernel_names import launched
from test_gpu_masked_prefix import check, masked_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("padding", [0, 64, 700, "holes"])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk,causal", [
    (3, 8, 8, 500, 8192, False), (1, 32, 8, 512, 8192, True), (1, 16, 16, 1280, 2400, True), (1, 16, 4, 1250, 2390, True), (2, 16, 16, 130, 5000, True),
    (6, 16, 4, 161, 4669, False)])
def test_two_groups(B, Hq, Hkv, Nq, Nk, causal, padding):
    q, k, v = masked_inputs(B, Hq, Hkv, Nq, Nk, 128, padding)
    print(f"launch split B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} causal={causal} {padding}", flush=True)
    (o, lse), names = launched(lambda: attn.rect_fwd(q, k, v, causal, 1 / math.sqrt(128)))
    kernel = f"attn_fwd_phase_kernel<128, {str(causal).lower()}, true, true, 2>"
    assert any(kernel in n for n in names) and any("attn_fwd_combine_kernel" in n for n in names), names
    check(o, lse, q, k, v, causal, 1 / math.sqrt(128))


@pytest.mark.parametrize("padding", [0, 64, "holes"])
@pytest.mark.parametrize("B,Hq,Hkv,Nq,Nk", [(13, 64, 8, 2, 1700), (16, 64, 16, 64, 1536), (25, 31, 31, 17, 129), (16, 64, 64, 1, 321)])
def test_few_rows(B, Hq, Hkv, Nq, Nk, padding):
    """Few rows under the causal mask at D = 64, with more workgroups than the phase kernel has places: with scratch the kernel of few rows,
    without it the phase kernel, whose bits do not depend on the number of heads."""
    q, k, v = masked_inputs(B, Hq, Hkv, Nq, Nk, 64, padding)
    scale = 1 / math.sqrt(64)
    print(f"launch few rows B{B} Hq{Hq} Hkv{Hkv} Nq{Nq} Nk{Nk} {padding}", flush=True)
    (o, lse), names = launched(lambda: attn.rect_fwd(q, k, v, True, scale))
    assert len(names) == 1 and "attn_fwd_kernel<64, true, true, false>" in names[0], names
    check(o, lse, q, k, v, True, scale)
    o, lse = torch.full_like(o, math.nan), torch.full_like(lse, math.nan)
    rc, names = launched(lambda: attn.tk_attn_fwd_rect(q, k, v, o, lse, B, Hq, Hkv, Nq, Nk, 64, True, scale))
    assert rc == attn.TK_OK and len(names) == 1 and "attn_fwd_phase_kernel" in names[0], names
    check(o, lse, q, k, v, True, scale)


@pytest.mark.parametrize("B,Hq,Nq,Nk", [(12, 64, 2, 1700), (16, 64, 65, 1700), (16, 64, 64, 64), (16, 65, 2, 1700)])
def test_other_rows(B, Hq, Nq, Nk):
    assert attn.tk_attn_fwd_scratch_bytes(B, Hq, Hq, Nq, Nk, 64, True) == 0
