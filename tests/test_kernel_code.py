"""What the compiler made of the kernels, read from the built library's gfx950 code (no GPU needed)."""
import os
import re
import struct
import subprocess

import pytest

from paper_2410_20399_amd import build

LLVM = "/opt/rocm/llvm/bin"


@pytest.fixture(scope="module")
def code_objects(tmp_path_factory):
    """The device code objects in the library's fat binary: one bundle per source, a table of (offset, size, target) each."""
    build.build(force=False)
    data = open(build.LIB, "rb").read()
    out = []
    for m in re.finditer(b"__CLANG_OFFLOAD_BUNDLE__", data):
        at, (count,) = m.end() + 8, struct.unpack_from("<Q", data, m.end())
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, at)
            target = data[at + 24:at + 24 + length].decode()
            at += 24 + length
            if "gfx950" in target and size:
                path = tmp_path_factory.mktemp("code") / f"{len(out)}.co"
                path.write_bytes(data[m.start() + offset:m.start() + offset + size])
                out.append(str(path))
    assert len(out) >= 5
    return out


def run(tool, *args):
    return subprocess.run([os.path.join(LLVM, tool), *args], check=True, capture_output=True, text=True).stdout


# The forward kernels at D = 64 hold three waves to a SIMD, 168 registers each.  What does not fit is kept from the prologue to
# the epilogue, and in the split ones beside the loop: its ordinary path touches no scratch memory.
SCRATCH = {"attn_fwd_phase_kernelILi64ELb1ELb1ELb0ELi1E": 8, "attn_fwd_phase_kernelILi64ELb1ELb1ELb1ELi1E": 20, "attn_fwd_phase_kernelILi64ELb0ELb1ELb1ELi1E": 16}


def test_scratch_memory(code_objects):
    """A spilled register's reload waits for every load before it, the prefetches of the loops among them."""
    kernels = {}
    for path in code_objects:
        for block in re.split(r"\n\s+- \.agpr_count", run("llvm-readelf", "--notes", path))[1:]:
            name = re.findall(r"\.name:\s+(\S+)", block)[-1]        # (after those of its arguments, if they have any)
            kernels[name] = int(re.search(r"\.private_segment_fixed_size:\s+(\d+)", block)[1])
    assert sum("attn_bwd_dkdv_wide_kernel" in n for n in kernels) == 8
    for name, size in kernels.items():
        assert size <= sum(most for part, most in SCRATCH.items() if part in name), (name, size)
