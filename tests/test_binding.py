"""The convenience functions of attn.py: what they refuse, and that they honour out= and stream=."""
import math
import os
import subprocess
import sys

import pytest
import torch

from paper_2410_20399_amd import attn


def test_tensors_that_are_not_on_the_gpu_are_refused():
    x = torch.zeros(1, 2, 128, 64, dtype=torch.bfloat16)
    with pytest.raises(ValueError):
        attn.attn_fwd(x, x, x, False, 1.0)
    with pytest.raises(ValueError):
        attn.gemm(x[0, 0], x[0, 0].t())
    with pytest.raises(TypeError):
        attn.rotary(None, x, x)


ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

# A library that stands in for the real one, and tensors without memory: the way from Python into the library, on the CPU.
STAND_IN = """
import sys, threading, time
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2410_20399_amd import attn
attn.load_library(sys.argv[1])
class Stream:
    cuda_stream = 0
with FakeTensorMode():
    a, b, c = (torch.empty(s, dtype=torch.bfloat16, device="cuda") for s in ((16, 64), (64, 24), (16, 24)))
"""


@pytest.fixture(scope="module")
def stand_in(tmp_path_factory):
    folder = tmp_path_factory.mktemp("stand_in")
    source, library = str(folder / "lib.c"), str(folder / "lib.so")
    with open(source, "w") as f:
        f.write("#include <unistd.h>\n")
        for name in attn.EXPORTS:
            f.write("int %s() { return 0; }\n" % name if name != "tk_gemm" else "int tk_gemm() { usleep(400000); return 0; }\n")
    subprocess.run(["gcc", "-shared", "-fPIC", source, "-o", library], check=True)

    def run(program):
        subprocess.run([sys.executable, "-c", STAND_IN + program, library], check=True, cwd=ROOT, timeout=120)
    return run


def test_the_library_that_was_loaded_is_the_one_that_is_called(stand_in):
    # (the real library refuses the missing memory)
    stand_in("assert attn.gemm(a, b, out=c, stream=Stream()) is not None\n")


def test_other_threads_run_while_a_call_is_in_the_library(stand_in):
    # (the stand-in stays in tk_gemm for 0.4 s, as a launch on a full queue does)
    stand_in("""
attn.gemm(a, b, out=c, stream=Stream())
awake = []
def wake():
    time.sleep(0.05)
    awake.append(time.monotonic())
thread = threading.Thread(target=wake)
thread.start()
attn.gemm(a, b, out=c, stream=Stream())
back = time.monotonic()
thread.join()
assert awake[0] < back - 0.1, (awake[0], back)
""")


def tensors(B, H, N, D, n=3):
    g = torch.Generator(device="cuda").manual_seed(N)
    return [torch.randn(B, H, N, D, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(n)]


@pytest.mark.gpu
def test_wrong_shapes_types_and_dimensions():
    q, k, v = tensors(2, 4, 128, 64)
    for bad in (k[:, :2].contiguous(), k[:, :, :64].contiguous(), k.float(), k.transpose(2, 3)):
        with pytest.raises(ValueError):
            attn.attn_fwd(q, bad, v, False, 0.125)
        with pytest.raises(ValueError):
            attn.attn_fwd(q, k, bad, False, 0.125)
    with pytest.raises(ValueError):
        attn.gqa_fwd(q, k[:, :2, :64].contiguous(), v[:, :2, :64].contiguous(), False, 0.125)
    with pytest.raises(ValueError):
        attn.decode(q, k, v, 0.125)
    o, lse = attn.attn_fwd(q, k, v, False, 0.125)
    with pytest.raises(ValueError):
        attn.attn_bwd(q, k, v, o, o, lse[:1].contiguous(), False, 0.125)
    with pytest.raises(attn.TkAttnError):
        attn.attn_fwd(q[..., :32].contiguous(), k[..., :32].contiguous(), v[..., :32].contiguous(), False, 0.125)
    with pytest.raises(attn.TkAttnError):
        attn.attn_bwd(q, k, v, o, o, lse, False, 0.125, workspace=torch.empty(16, dtype=torch.uint8, device="cuda"))
    with pytest.raises(attn.TkAttnError):
        attn.gemm(torch.zeros(8, 12, dtype=torch.bfloat16, device="cuda"), torch.zeros(12, 8, dtype=torch.bfloat16, device="cuda"))


@pytest.mark.gpu
def test_out_and_stream_are_honoured():
    B, H, N, D = 1, 2, 300, 128
    q, k, v, d_o = tensors(B, H, N, D, 4)
    scale = 1 / math.sqrt(D)
    o, lse = attn.attn_fwd(q, k, v, True, scale)
    grads = attn.attn_bwd(q, k, v, o, d_o, lse, True, scale)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    o2, lse2 = torch.empty_like(o), torch.empty_like(lse)
    grads2 = tuple(torch.empty_like(q) for _ in range(3))
    workspace = attn.alloc_bwd_workspace(B, H, N, D)
    torch.cuda.synchronize()
    assert attn.attn_fwd(q, k, v, True, scale, out=(o2, lse2), stream=side)[0].data_ptr() == o2.data_ptr()
    attn.attn_bwd(q, k, v, o2, d_o, lse2, True, scale, workspace=workspace, out=grads2, stream=side)
    side.synchronize()          # (nothing else is waited for: the work was on this stream)
    assert torch.equal(o, o2) and torch.equal(lse, lse2)
    assert all(torch.equal(a, b) for a, b in zip(grads, grads2))
    with torch.cuda.stream(side):
        o3, _ = attn.attn_fwd(q, k, v, True, scale)
    side.synchronize()
    assert torch.equal(o, o3)


@pytest.mark.gpu
@pytest.mark.parametrize("D", [64, 128])
def test_own_workspace_belongs_to_the_stream_of_the_call(D):
    """A backward call without a workspace, on a stream that is still busy: what the current stream allocates right after
    the call is not the memory that the call has yet to write."""
    B, H, N = 1, 4, 1024
    q, k, v, d_o = tensors(B, H, N, D, 4)
    scale = 1 / math.sqrt(D)
    o, lse = attn.attn_fwd(q, k, v, True, scale)
    want = attn.attn_bwd(q, k, v, o, d_o, lse, True, scale)
    n = attn.alloc_bwd_workspace(B, H, N, D).numel()
    a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
    c = torch.empty_like(a)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    for call in (lambda: attn.attn_bwd(q, k, v, o, d_o, lse, True, scale, stream=side),
                 lambda: attn.gqa_bwd(q, k, v, o, d_o, lse, True, scale, stream=side),
                 lambda: attn.rect_bwd(q, k, v, o, d_o, lse, True, scale, stream=side)):
        for _ in range(60):
            attn.gemm(a, a, out=c, stream=side)         # (about 50 ms, which the backward waits behind)
        got = call()
        junk = [torch.full((n,), 0x5A, dtype=torch.uint8, device="cuda") for _ in range(4)]
        torch.cuda.current_stream().synchronize()
        assert not side.query(), "the other stream was to be busy until here"
        side.synchronize()
        assert all(bool((t == 0x5A).all()) for t in junk), "the call wrote memory that was no longer its own"
        assert all(torch.equal(x, y) for x, y in zip(got, want))
        del junk


@pytest.mark.gpu
@pytest.mark.skipif(torch.cuda.device_count() < 2, reason="needs a device that is not the current one")
def test_scratch_belongs_to_the_stream_of_another_device():
    """The tensors and the stream are the second device's, the first is the current one."""
    with torch.cuda.device(1):
        g = torch.Generator(device="cuda").manual_seed(3)
        q, d_o = (torch.randn(1, 8, 512, 128, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        k, v = (torch.randn(1, 2, 4096, 128, generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(2))
        o, lse = attn.rect_fwd(q, k, v, True, 0.1)
        want = (o, lse, *attn.rect_bwd(q, k, v, o, d_o, lse, True, 0.1))
        a = torch.randn(8192, 8192, device="cuda", dtype=torch.bfloat16)
        c = torch.empty_like(a)
        side = torch.cuda.Stream()
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
    for call in (lambda: attn.rect_fwd(q, k, v, True, 0.1, stream=side), lambda: attn.rect_bwd(q, k, v, o, d_o, lse, True, 0.1, stream=side)):
        for _ in range(20):
            attn.gemm(a, a, out=c, stream=side)
        got = call()
        junk = [torch.full((n << 20,), 0x5A, dtype=torch.uint8, device="cuda:1") for n in (1, 4, 16, 64)]
        torch.cuda.current_stream(1).synchronize()
        side.synchronize()
        assert all(bool((t == 0x5A).all()) for t in junk)
        assert all(torch.equal(x, y) for x, y in zip(got, want[:2] if len(got) == 2 else want[2:]))


@pytest.mark.gpu
def test_backward_refuses_q_of_another_rank():
    q, k, v = tensors(2, 4, 128, 64)
    o, lse = attn.attn_fwd(q, k, v, False, 0.125)
    for bad in (q[0].contiguous(), q[None].contiguous()):
        for f in (attn.attn_bwd, attn.gqa_bwd, attn.rect_bwd):
            with pytest.raises(ValueError):
                f(bad, k, v, o, o, lse, False, 0.125)


@pytest.mark.gpu
def test_outputs_and_workspaces_that_do_not_fit_are_refused():
    """Whatever the kernels would write to is looked at before anything is launched."""
    q, k, v, d_o = tensors(1, 4, 256, 64, 4)
    o, lse = attn.attn_fwd(q, k, v, False, 0.125)
    workspace = attn.alloc_bwd_workspace(1, 4, 256, 64)
    new = lambda *shape: torch.empty(shape, dtype=torch.bfloat16, device="cuda")
    wrong = (new(1, 4, 255, 64), new(1, 4, 256, 64).float(), new(1, 4, 256, 64).cpu(), new(1, 4, 64, 256).transpose(2, 3), new(4 * 256 * 64))
    for bad in wrong:
        for i in range(3):
            out = [torch.empty_like(q) for _ in range(3)]
            out[i] = bad
            with pytest.raises(ValueError):
                attn.attn_bwd(q, k, v, o, d_o, lse, False, 0.125, workspace=workspace, out=out)
        with pytest.raises(ValueError):
            attn.attn_fwd(q, k, v, False, 0.125, out=(bad, lse))
        with pytest.raises(ValueError):
            attn.rotary(q, new(256, 32), new(256, 32), out=bad)
    for out in ((None, None, None), (None, torch.empty_like(k), torch.empty_like(v)), (torch.empty_like(q), None, None), 3):
        with pytest.raises((TypeError, attn.TkAttnError)):
            attn.attn_bwd(q, k, v, o, d_o, lse, False, 0.125, workspace=workspace, out=out)
    for out in ((None, None), (None, lse), (o, None)):
        with pytest.raises((TypeError, AttributeError)):
            attn.attn_fwd(q, k, v, False, 0.125, out=out)
    for out in ((o,), (o, lse, lse)):
        with pytest.raises(ValueError):
            attn.attn_fwd(q, k, v, False, 0.125, out=out)
    for bad in (workspace.cpu(), workspace[::2], torch.zeros(1, dtype=torch.uint8, device="cuda").expand(1 << 20), torch.zeros(1 << 20, dtype=torch.uint8)):
        with pytest.raises(ValueError):
            attn.attn_bwd(q, k, v, o, d_o, lse, False, 0.125, workspace=bad)
        with pytest.raises(ValueError):
            attn.decode(q[:, :, :1].contiguous(), k, v, 0.125, workspace=bad)
    with pytest.raises(TypeError):
        attn.attn_bwd(q, k, v, o, d_o, lse, False, 0.125, workspace=1 << 20)
    a, b = new(16, 64), new(64, 24)
    for bad in (new(16, 23), new(24, 16), new(16, 24).float(), new(16, 24).cpu(), new(24, 16).t(), new(15, 24), new(16 * 24)):
        with pytest.raises(ValueError):
            attn.gemm(a, b, out=bad)


@pytest.mark.gpu
def test_without_memory_for_scratch_a_call_does_without():
    """The scratch of a split is no more than an aid: a process at its memory limit gets the unsplit results."""
    B, Hq, Hkv, D, scale = 1, 32, 8, 64, 0.125
    torch.cuda.empty_cache()            # (no large block of an earlier test, of which a part would be left over)
    g = torch.Generator(device="cuda").manual_seed(5)
    new = lambda h, n: torch.randn(B, h, n, D, generator=g, device="cuda", dtype=torch.bfloat16)
    q, k, v = new(Hq, 1024), new(Hkv, 8192), new(Hkv, 8192)
    q2, k2, v2, d_o = new(Hq, 2048), new(Hkv, 2048), new(Hkv, 2048), new(Hq, 2048)
    assert attn.tk_attn_fwd_scratch_bytes(B, Hq, Hkv, 1024, 8192, D, True) > 16 << 20
    workspace = torch.empty(attn.tk_attn_bwd_workspace_bytes(B, Hq, 2048, D), dtype=torch.uint8, device="cuda")
    assert attn.tk_attn_bwd_scratch_bytes(B, Hq, Hkv, 2048, 2048, D, True, workspace.numel()) > 16 << 20
    o, lse = torch.empty_like(q), torch.empty(B, Hq, 1024, device="cuda")
    assert attn.tk_attn_fwd_rect(q, k, v, o, lse, B, Hq, Hkv, 1024, 8192, D, True, scale) == attn.TK_OK
    o2, lse2 = attn.gqa_fwd(q2, k2, v2, True, scale)
    grads = tuple(torch.empty_like(t) for t in (q2, k2, v2))
    assert attn.tk_attn_bwd_rect(q2, k2, v2, o2, d_o, lse2, *grads, B, Hq, Hkv, 2048, 2048, D, True, scale, workspace, workspace.numel()) == attn.TK_OK
    torch.cuda.synchronize()
    keep = [torch.empty_like(t) for t in (o, lse, *grads)]      # (memory for the results, given back to the pool)
    torch.cuda.empty_cache()
    del keep
    total = torch.cuda.get_device_properties(0).total_memory
    try:
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (1 << 20)) / total)
        with pytest.raises(torch.OutOfMemoryError):
            torch.empty(32 << 20, dtype=torch.uint8, device="cuda")
        got = attn.rect_fwd(q, k, v, True, scale)
        got_grads = attn.gqa_bwd(q2, k2, v2, o2, d_o, lse2, True, scale, workspace)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(got[0], o) and torch.equal(got[1], lse)
    assert all(torch.equal(x, y) for x, y in zip(got_grads, grads))
