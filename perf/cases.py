"""Performance cases: the calls a program built on this package makes, over the sizes it makes them with.

Seven kinds of call, all through the public functions of ``paper_2410_20399_amd.attn``:

  fwd      attn_fwd: inference of a multi-head layer (no gradients)
  prefill  rotary on Q and K, then gqa_fwd with the causal mask: a prompt of a grouped-query decoder
  chunk    rect_fwd with the causal mask: a chunk of a prompt against the keys already in the history
  decode   one new token per sequence against its key/value history
  train    attn_fwd or gqa_fwd, then the matching backward: one layer of a training step
  cross    rect_fwd and rect_bwd without a mask: cross-attention in training
  gemm     the projections around the attention

``listed()`` are fixed sizes: the benchmark's own workloads and the odd sizes of the tests or generic ones;
``draw(rng)`` gives further sizes of the same ranges.
"""
import math

import torch

from paper_2410_20399_amd import attn

# the work of the largest listed case (forward and backward, causal, B16 H16 N4096 D128): no drawn case is larger
MAX_FLOPS = 14.0 * 16 * 16 * (4096 * 4097 // 2) * 128
MAX_BYTES = 2.0e9


def listed():
    return [
        # one tile of work: what a call costs before there is anything to do (the first forward workload)
        dict(name="fwd_one_tile", kind="fwd", B=1, Hq=1, Hkv=1, Nq=128, Nk=128, D=64, causal=False),
        # an encoder layer on a batch of ordinary sequences, head dimension 64 (the second forward workload)
        dict(name="fwd_encoder_d64", kind="fwd", B=16, Hq=16, Hkv=16, Nq=1024, Nk=1024, D=64, causal=False),
        # one user's prompt, of no particular length, through a grouped-query layer
        dict(name="prefill_ragged", kind="prefill", B=1, Hq=32, Hkv=8, Nq=3001, Nk=3001, D=128, causal=True),
        # the last chunk of a long prompt: 512 queries that see 8192 keys
        dict(name="chunk_512_of_8192", kind="chunk", B=1, Hq=32, Hkv=8, Nq=512, Nk=8192, D=128, causal=True),
        # serving a batch with long histories (the benchmark's decode workload)
        dict(name="decode_batch16", kind="decode", B=16, Hq=32, Hkv=8, Nq=1, Nk=8192, D=128, causal=False),
        # one user, a short history: latency
        dict(name="decode_single", kind="decode", B=1, Hq=32, Hkv=8, Nq=1, Nk=2000, D=128, causal=False),
        # the benchmark's headline workload: one training layer
        dict(name="train_d128", kind="train", B=16, Hq=16, Hkv=16, Nq=4096, Nk=4096, D=128, causal=True),
        # the same with head dimension 64
        dict(name="train_d64", kind="train", B=16, Hq=16, Hkv=16, Nq=4096, Nk=4096, D=64, causal=True),
        # fine-tuning on short samples: a small batch, grouped heads, a length that is no multiple of anything
        dict(name="train_gqa_ragged", kind="train", B=2, Hq=16, Hkv=4, Nq=1001, Nk=1001, D=128, causal=True),
        # a decoder that attends to an encoder's output of another, odd length
        dict(name="cross_1000x300_d64", kind="cross", B=4, Hq=16, Hkv=16, Nq=1000, Nk=300, D=64, causal=False),
        # the fused QKV projection of a 2048-wide layer for about a thousand tokens
        dict(name="gemm_qkv_1000", kind="gemm", M=1000, N=6144, K=2048),
        # the benchmark's GEMM workload
        dict(name="gemm_8192", kind="gemm", M=8192, N=8192, K=8192),
    ]


def _log_int(rng, lo, hi):
    """A whole number between lo and hi, spread over its logarithm; every second one a multiple of the power of two below it."""
    n = min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))
    if rng.random() < 0.5:
        unit = min(128, 1 << (n.bit_length() - 1))
        n = max(lo, n // unit * unit)
    return n


def _draw_once(rng):
    kind = rng.choice(["fwd", "prefill", "chunk", "decode", "train", "train", "cross", "gemm"])
    if kind == "gemm":
        return dict(kind=kind, M=_log_int(rng, 16, 8192), N=8 * _log_int(rng, 32, 1024), K=8 * _log_int(rng, 32, 1024))
    D = rng.choice([64, 128])
    causal = kind in ("prefill", "chunk") or (kind in ("fwd", "train") and rng.random() < 0.5)
    grouped = kind in ("prefill", "chunk", "decode") or (kind == "train" and rng.random() < 0.5)
    Hkv = rng.choice([1, 2, 4, 8]) if grouped else rng.choice([4, 8, 12, 16])
    Hq = Hkv * (rng.choice([2, 4, 8]) if grouped else 1)
    B = _log_int(rng, 1, 16)
    if kind == "fwd":
        Nq = Nk = _log_int(rng, 64, 4096)
    elif kind == "prefill":
        B, Nq = min(B, 4), _log_int(rng, 128, 16384)
        Nk = Nq
    elif kind == "chunk":
        B, Nq = min(B, 4), _log_int(rng, 32, 1024)
        Nk = Nq + _log_int(rng, 128, 16384)
    elif kind == "decode":
        B, Nq, Nk = _log_int(rng, 1, 64), 1, _log_int(rng, 128, 65536)
    elif kind == "train":
        Nq = Nk = _log_int(rng, 256, 16384)
    else:
        Nq, Nk = _log_int(rng, 128, 4096), _log_int(rng, 64, 2048)
    return dict(kind=kind, B=B, Hq=Hq, Hkv=Hkv, Nq=Nq, Nk=Nk, D=D, causal=causal)


def draw(rng):
    while True:
        case = _draw_once(rng)
        w = work(case)
        if w["flops"] <= MAX_FLOPS and w["bytes"] <= MAX_BYTES:
            return case


def _pairs(case):
    """(query, key) pairs of one head that the mask keeps."""
    Nq, Nk = case["Nq"], case["Nk"]
    return Nq * (Nk - Nq) + Nq * (Nq + 1) // 2 if case["causal"] else Nq * Nk


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.bfloat16)

    kind = case["kind"]
    if kind == "gemm":
        return dict(kind=kind, a=normal(case["M"], case["K"]), b=normal(case["K"], case["N"]))
    B, Hq, Hkv, Nq, Nk, D = (case[n] for n in ("B", "Hq", "Hkv", "Nq", "Nk", "D"))
    s = dict(kind=kind, causal=case["causal"], grouped=Hkv != Hq, scale=1 / math.sqrt(D),
             q=normal(B, Hq, Nq, D), k=normal(B, Hkv, Nk, D), v=normal(B, Hkv, Nk, D))
    if kind == "prefill":
        angle = torch.arange(Nq, device="cuda", dtype=torch.float32)[:, None] * torch.logspace(0, -4, D // 2, device="cuda")
        s["sin"], s["cos"] = angle.sin().to(torch.bfloat16), angle.cos().to(torch.bfloat16)
    if kind in ("train", "cross"):          # the incoming gradient, and the workspace that a training loop keeps
        s["d_o"] = normal(B, Hq, Nq, D)
        s["workspace"] = attn.alloc_bwd_workspace(B, Hq, Nq, D, Nk=Nk)
    if kind == "decode":                    # (kept by a serving loop, too)
        s["workspace"] = torch.empty(attn.tk_attn_decode_workspace_bytes(B, Hq, Hkv, Nk, D), dtype=torch.uint8, device="cuda")
    return s


def run(state):
    kind = state["kind"]
    if kind == "gemm":
        return attn.gemm(state["a"], state["b"])
    q, k, v, causal, scale = state["q"], state["k"], state["v"], state["causal"], state["scale"]
    if kind == "fwd":
        return attn.attn_fwd(q, k, v, causal, scale)
    if kind == "prefill":
        q, k = attn.rotary(q, state["sin"], state["cos"]), attn.rotary(k, state["sin"], state["cos"])
        o, lse = attn.gqa_fwd(q, k, v, causal, scale)
        return o, lse, k                    # (k goes into the key/value history)
    if kind == "chunk":
        return attn.rect_fwd(q, k, v, causal, scale)
    if kind == "decode":
        return attn.decode(q, k, v, scale, workspace=state["workspace"])
    if kind == "cross":
        o, lse = attn.rect_fwd(q, k, v, causal, scale)
        return o, lse, *attn.rect_bwd(q, k, v, o, state["d_o"], lse, causal, scale, workspace=state["workspace"])
    forward, backward = (attn.gqa_fwd, attn.gqa_bwd) if state["grouped"] else (attn.attn_fwd, attn.attn_bwd)
    o, lse = forward(q, k, v, causal, scale)
    return o, lse, *backward(q, k, v, o, state["d_o"], lse, causal, scale, workspace=state["workspace"])


def work(case):
    kind = case["kind"]
    if kind == "gemm":
        M, N, K = case["M"], case["N"], case["K"]
        return {"bytes": 2.0 * (M * K + K * N + M * N), "flops": 2.0 * M * N * K}
    B, Hq, Hkv, Nq, Nk, D = (case[n] for n in ("B", "Hq", "Hkv", "Nq", "Nk", "D"))
    q_bytes, kv_bytes, lse_bytes = 2.0 * B * Hq * Nq * D, 2.0 * B * Hkv * Nk * D, 4.0 * B * Hq * Nq
    pairs = float(B * Hq) * _pairs(case)
    n_bytes, flops = 2 * q_bytes + 2 * kv_bytes + lse_bytes, 4.0 * D * pairs
    if kind == "prefill":                   # the two tables in, the rotated keys out
        n_bytes += 2.0 * Nq * D + kv_bytes
        flops += 3.0 * (q_bytes + kv_bytes) / 2
    if kind in ("train", "cross"):          # the incoming gradient in, three gradients out; five products per pair
        n_bytes += 2 * q_bytes + 2 * kv_bytes
        flops += 10.0 * D * pairs
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # Measured against the same calls in float64, over these cases and two dozen drawn ones: one rounding to bf16
    # leaves 1.7e-3 in a GEMM, the rounding of P to bf16 as well 2.0e-3 to 2.4e-3 in O, that of dS and of the O inside
    # Delta 2.3e-3 to 2.5e-3 in the gradients.  Stated: four times that.
    # Largest single element: 4e-3 in a GEMM (half a bf16 ulp), 3e-2 in O, 0.13 in a causal gradient, where
    # dP - Delta cancels in the rows of the first few keys.
    if case["kind"] == "gemm":
        return {"rel": 7e-3, "max": 1.6e-2}
    if case["kind"] in ("train", "cross"):
        return {"rel": 1e-2, "max": 0.5}
    return {"rel": 1e-2, "max": 0.12}
