"""GPU parity for the bf16 GEMM against the fp64 oracle.

Tolerance: fp32 accumulation of K bf16 products and one rounding to bf16.  Per element the error
is at most half a bf16 ulp of the result (2^-8 |ref|) plus the fp32 accumulation error, bounded
here by K * 2^-24 * sum_k |a_ik b_kj| <= K * 2^-24 * (a generous 4 * sqrt(K)) for unit-variance data."""
import math

import numpy as np
import pytest
import torch

from oracle import attn_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def attn():
    from paper_2410_20399_amd import attn as a
    a.load_library()
    return a


def make(M, N, K, seed):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(M, K, generator=g).to(torch.bfloat16), torch.randn(K, N, generator=g).to(torch.bfloat16)


def tol(ref, K):
    return 2.0 ** -8 * np.abs(ref) + K * 2.0 ** -24 * 4 * np.sqrt(K) + 1e-6


@pytest.mark.parametrize("M,N,K", [(256, 256, 64), (256, 512, 128), (512, 256, 192), (768, 1280, 320), (256, 256, 2048)])
def test_gemm_small_full(attn, M, N, K):
    a, b = make(M, N, K, 840 + M + N + K)
    print(f"launch gemm M{M} N{N} K{K}", flush=True)
    c = attn.gemm(a.cuda(), b.cuda())
    torch.cuda.synchronize()
    ref = orc.gemm(a.double().numpy(), b.double().numpy())
    err = np.abs(c.cpu().double().numpy() - ref)
    assert (err <= tol(ref, K)).all(), float((err - tol(ref, K)).max())


@pytest.mark.parametrize("M,N,K", [(1, 8, 8), (5, 24, 40), (255, 264, 72), (257, 248, 200), (300, 520, 1000), (1000, 1000, 1000),
                                   (256, 256, 56), (513, 256, 64), (256, 776, 128)])
def test_gemm_edge_tiles(attn, M, N, K):
    """Shapes that are not multiples of any tile: every element against the oracle, and the
    memory after C untouched (rows and columns past the end are masked, not clipped by luck)."""
    a, b = make(M, N, K, 1840 + M + N + K)
    print(f"launch gemm edge M{M} N{N} K{K}", flush=True)
    guard = 4096
    buf = torch.full((M * N + guard,), 77.0, dtype=torch.bfloat16, device="cuda")
    c = buf[:M * N].view(M, N)
    attn.gemm(a.cuda(), b.cuda(), out=c)
    torch.cuda.synchronize()
    assert bool((buf[M * N:] == 77.0).all()), "wrote past the end of C"
    ref = orc.gemm(a.double().numpy(), b.double().numpy())
    err = np.abs(c.cpu().double().numpy() - ref)
    assert np.isfinite(err).all()
    assert (err <= tol(ref, K)).all(), float((err - tol(ref, K)).max())


def test_gemm_full_size_sampled_and_reproducible(attn):
    M = N = K = 8192
    a, b = make(M, N, K, 8192)
    print("launch gemm 8192^3", flush=True)
    ad, bd = a.cuda(), b.cuda()
    c1 = attn.gemm(ad, bd)
    c2 = attn.gemm(ad, bd)
    torch.cuda.synchronize()
    assert torch.equal(c1, c2)
    rng = np.random.default_rng(7)
    rows = np.concatenate([rng.integers(0, M, 4000), [0, M - 1, 255, 256]])
    cols = np.concatenate([rng.integers(0, N, 4000), [0, N - 1, 256, 255]])
    ref = orc.gemm_elements(a.double().numpy(), b.double().numpy(), rows, cols)
    got = c1.cpu().double().numpy()[rows, cols]
    err = np.abs(got - ref)
    assert (err <= tol(ref, K)).all(), float((err - tol(ref, K)).max())
    # every 256 x 256 tile is touched: no tile left at its initial value
    c3 = torch.full((M, N), 12345.0, dtype=torch.bfloat16, device="cuda")
    attn.gemm(ad, bd, out=c3)
    torch.cuda.synchronize()
    assert torch.equal(c3, c1)


# One or two sizes for each tile shape the launcher chooses from (256x256 .. 32x64, K split in 2 and in 4): ragged
# rows and columns, a K that ends inside a step, fewer steps than ring stages, K shares of unequal length.
@pytest.mark.parametrize("M,N,K", [(3101, 3888, 72), (2731, 5000, 328), (2657, 3416, 200), (3352, 3288, 24), (1488, 4040, 264),
                                   (1351, 5488, 392), (2455, 1808, 328), (863, 5192, 72), (1425, 1464, 456), (1974, 1152, 8),
                                   (1641, 4944, 200), (1010, 1104, 136), (805, 8, 24), (238, 16, 24), (2068, 200, 72),
                                   (599, 840, 584), (97, 48, 96), (22, 216, 328), (1, 320, 256), (59, 24, 424), (14, 352, 1096)])
def test_gemm_every_tile_shape(attn, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.randn(M, K, generator=g, device="cuda", dtype=torch.bfloat16)
    b = torch.randn(K, N, generator=g, device="cuda", dtype=torch.bfloat16)
    print(f"launch gemm M{M} N{N} K{K}", flush=True)
    guard = 4096
    buf = torch.full((M * N + guard,), 77.0, dtype=torch.bfloat16, device="cuda")
    attn.gemm(a, b, out=buf[:M * N].view(M, N))
    torch.cuda.synchronize()
    assert bool((buf[M * N:] == 77.0).all()), "wrote past the end of C"
    ref = a.cpu().double().numpy() @ b.cpu().double().numpy()
    err = np.abs(buf[:M * N].view(M, N).cpu().double().numpy() - ref)
    assert np.isfinite(err).all()
    assert (err <= tol(ref, K)).all(), float((err - tol(ref, K)).max())


# Matrices whose rows within one tile lie up to and beyond 4 GiB apart: wide B (a step has 64 of its rows) and long rows
# of A, on both sides of the line, where the lanes' offsets no longer fit 32 bits.
@pytest.mark.parametrize("M,N,K", [(16, 20_000_000, 64), (1, 33_554_432, 64), (1, 34_200_008, 72), (40, 36_000_008, 64), (250, 34_500_008, 64), (300, 35_000_000, 128),
                                   (32, 8, 40_000_000), (32, 8, 69_400_008), (200, 72, 34_000_000)])
def test_gemm_offsets_beyond_32_bits(attn, M, N, K):
    g = torch.Generator(device="cuda").manual_seed(M + N + K)
    a = torch.empty(M, K, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    b = torch.empty(K, N, device="cuda", dtype=torch.bfloat16).normal_(generator=g)
    print(f"launch gemm M{M} N{N} K{K}", flush=True)
    c = attn.gemm(a, b)
    torch.cuda.synchronize()
    cols = torch.arange(N)
    if N > 1600:
        cols = torch.cat([cols[:300], torch.randint(N, (1000,), generator=torch.Generator().manual_seed(N)), cols[-300:]])
    cols = cols.cuda()
    ref = torch.zeros(M, len(cols), device="cuda", dtype=torch.float64)
    for k0 in range(0, K, 1 << 20):
        ref += a[:, k0:k0 + (1 << 20)].double() @ b[k0:k0 + (1 << 20), cols].double()
    err = (c[:, cols].double() - ref).abs()
    # half a bf16 ulp, and the fp32 sums: up to K roundings of partial sums of the size sqrt(k), which add up like a random
    # walk to less than 0.3 * 2^-24 * K (rms)
    bound = 2.0 ** -8 * ref.abs() + 2.0 ** -24 * K + 1e-5 * math.sqrt(K)
    assert bool((err <= bound).all()), float((err - bound).max())
