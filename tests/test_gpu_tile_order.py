"""GPU: every (head, query tile) of a launch is computed exactly once, whatever the number of heads.

The forward walks groups of heads together, last tiles first; the group size depends on the number of heads and
tiles, and the last group may be smaller or no multiple of 8.  A head's result does not depend on its neighbours,
so each head of a batched call must equal the same head run alone, bit for bit, and nothing may stay unwritten.
"""
import math

import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("causal", [True, False])
@pytest.mark.parametrize("B,H,N,D", [(1, 9, 300, 64), (3, 7, 1500, 128), (2, 13, 257, 128), (1, 70, 700, 64), (1, 24, 128, 64),
                                     (2, 20, 4000, 64),
                                     # no divisor of an XCD's heads near the group: the next one, one group and three; equal groups
                                     (4, 14, 1832, 64), (3, 24, 4224, 64), (3, 88, 312, 64),
                                     # the same with the larger groups of D = 64
                                     (8, 13, 2950, 64), (8, 9, 11000, 64), (8, 89, 312, 64)])
def test_every_tile_once(B, H, N, D, causal):
    g = torch.Generator().manual_seed(7 * N + H)
    q, k, v = (torch.randn(B, H, N, D, generator=g).to(torch.bfloat16).cuda() for _ in range(3))
    o = torch.full_like(q, float("nan"))
    lse = torch.full((B, H, N), float("nan"), dtype=torch.float32, device="cuda")
    print(f"launch order B{B} H{H} N{N} D{D} causal={causal}", flush=True)
    attn.attn_fwd(q, k, v, causal, 1 / math.sqrt(D), out=(o, lse))
    for b in range(B):
        for h in range(H):
            one = tuple(t[b:b + 1, h:h + 1].contiguous() for t in (q, k, v))
            o1, l1 = attn.attn_fwd(*one, causal, 1 / math.sqrt(D))
            assert torch.equal(o[b, h], o1[0, 0]) and torch.equal(lse[b, h], l1[0, 0]), (b, h)
