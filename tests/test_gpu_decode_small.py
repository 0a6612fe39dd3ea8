"""GPU: decode calls small enough that every workgroup has a compute unit of its own, with four waves sharing the keys.

Histories that end inside each wave's 32 keys, one trip and several, one split and many, groups of 1 to 32 heads, and the
first group that is too large.  Against the fp64 oracle with the bounds of the forward.
"""
import math

import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc
from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,Nk", [(1, 1, 1, 31), (2, 4, 2, 33), (1, 8, 2, 65), (1, 32, 1, 97), (1, 33, 1, 700), (3, 6, 3, 255),
                                         (1, 8, 2, 256), (1, 4, 4, 513), (1, 32, 8, 2000), (1, 2, 1, 40001)])
def test_small_decode(B, Hq, Hkv, Nk, D):
    g = torch.Generator().manual_seed(Nk + Hq + D)
    q, k, v = (torch.randn(B, h, n, D, generator=g).to(torch.bfloat16) for h, n in ((Hq, 1), (Hkv, Nk), (Hkv, Nk)))
    scale = 1 / math.sqrt(D)
    print(f"launch decode B{B} Hq{Hq} Hkv{Hkv} Nk{Nk} D{D}", flush=True)
    o, lse = attn.decode(q.cuda(), k.cuda(), v.cuda(), scale)
    torch.cuda.synchronize()
    o_ref, lse_ref = orc.rect_fwd(*(t.double().numpy() for t in (q, k, v)), False, scale)
    err = np.abs(o.double().cpu().numpy() - o_ref)
    assert err.max() <= 2e-2 and err.mean() <= 2e-3, (err.max(), err.mean())
    assert np.abs(lse.double().cpu().numpy() - lse_ref).max() <= 1e-3
