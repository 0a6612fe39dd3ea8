"""GPU: the matrix product's stream along K, around the lengths at which its loops begin and end.

Whole numbers of at most 4: every sum is exact in fp32, so that each element has to be the exact product rounded to bf16.
"""
import pytest
import torch

from paper_2410_20399_amd import attn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [64, 120, 128, 136, 192, 248, 256, 328, 448, 568, 840, 1024, 1088])
@pytest.mark.parametrize("M,N", [(3000, 3000), (2900, 2304), (1000, 6144), (3000, 1536), (1100, 2000), (300, 1000), (600, 64), (64, 512), (16, 304)])
def test_gemm_steps(M, N, K):
    g = torch.Generator(device="cuda").manual_seed(K)
    a, b = (torch.randint(-4, 5, shape, generator=g, device="cuda").to(torch.bfloat16) for shape in ((M, K), (K, N)))
    print(f"launch gemm M{M} N{N} K{K}", flush=True)
    c = attn.gemm(a, b)
    assert torch.equal(c, (a.float() @ b.float()).to(torch.bfloat16))
