"""GPU: split forward calls with workgroups of 256 query rows (D = 128): lengths that end inside a tile and inside a wave, splits that
lie wholly beyond the diagonal of a query tile, groups of heads, keys that the caller masks.  Checked in fp64 as the other split calls.
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
