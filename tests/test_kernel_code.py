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


# The 256-key dK/dV kernel issues the products that its accumulators take as inline assembly, for which the compiler keeps none of the
# distances that the matrix pipe wants (in issued instructions, s_nop n counting n + 1): two from a vector instruction that writes an
# operand to the product, 18 from the product to whatever else reads its accumulator, products of the same accumulator excepted.
OPERAND_DISTANCE, RESULT_DISTANCE = 2, 18


def registers(text):
    """{(file, number)} of the vector (v) and accumulator (a) registers that an operand text names"""
    out = set()
    for file, first, last, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))", text):
        out |= {(file, n) for n in range(int(first or one), int(last or one) + 1)}
    return out


def parse(listing):
    """Instructions of one function of llvm-objdump's listing: (name, operands, address, target of a branch or None)"""
    out, start = [], None
    for line in listing.splitlines():
        m = re.match(r"\s+(\S+)\s*(.*?)\s*// ([0-9A-F]+):[^<]*(?:<[^>]*?\+0x([0-9a-f]+)>)?", line)
        if m:
            address = int(m[3], 16)
            start = address if start is None else start
            target = start + int(m[4] or "0", 16) if "branch" in m[1] else None
            out.append((m[1], m[2], address, target))
    return out


def violations(code):
    at = {address: i for i, (_, _, address, _) in enumerate(code)}
    before = [[] for _ in code]                     # indices of the instructions that may run right before
    for i, (name, _, _, target) in enumerate(code):
        if i + 1 < len(code) and name not in ("s_branch", "s_endpgm"):
            before[i + 1].append(i)
        if target is not None:
            before[at[target]].append(i)
    uses = []                                       # (registers written, registers read)
    for name, operands, _, _ in code:
        first, _, rest = operands.partition(",")
        stores = name.startswith(("ds_write", "global_store", "buffer_store", "scratch_store", "flat_store"))
        uses.append((set(), registers(operands)) if stores else (registers(first), registers(rest)))
    product = [name.startswith("v_mfma") and operands.startswith("a[") for name, operands, _, _ in code]

    def reached_within(i, distance, wrong):
        """an instruction less than `distance` wait states ahead of i for which wrong() holds"""
        seen, todo = {}, [(p, distance) for p in before[i]]
        while todo:
            p, left = todo.pop()
            if left <= 0 or seen.get(p, 0) >= left:
                continue
            seen[p] = left
            if wrong(p):
                return p
            name, operands = code[p][:2]
            left -= int(operands, 0) + 1 if name == "s_nop" else 1
            todo += [(q, left) for q in before[p]]
        return None

    out = []
    for i, (name, _, _, _) in enumerate(code):
        written, read = uses[i]
        if product[i]:
            p = reached_within(i, OPERAND_DISTANCE, lambda p: code[p][0].startswith("v_") and not product[p] and uses[p][0] & read)
        elif any(file == "a" for file, _ in read):
            p = reached_within(i, RESULT_DISTANCE, lambda p: product[p] and uses[p][0] & read)
        else:
            continue
        if p is not None:
            out.append((code[p][:3], code[i][:3]))
    return out


def test_matrix_instruction_distances(code_objects):
    listings = [text for path in code_objects for text in re.split(r"\n(?=[0-9a-f]{16} <)", run("llvm-objdump", "-d", path)) if "attn_bwd_dkdv_wide_kernel" in text.split("\n")[0]]
    assert len(listings) == 8
    for text in listings:
        code = parse(text)
        assert sum(name.startswith("v_mfma") and operands.startswith("a[") for name, operands, _, _ in code) >= 64
        assert not violations(code), (text.split("\n")[0], violations(code)[:4])


@pytest.mark.parametrize("lines,wrong", [
    (["v_mul_f32_e32 v5, v1, v2", "s_nop 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"], True),
    (["v_mul_f32_e32 v5, v1, v2", "s_nop 1", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"], False),
    (["v_accvgpr_write_b32 a3, 0", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"], True),
    (["v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "s_nop 15", "v_accvgpr_read_b32 v0, a15"], True),
    (["v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "s_nop 15", "s_nop 1", "v_accvgpr_read_b32 v0, a15"], False),
    (["v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "s_nop 7", "global_store_dwordx4 v[0:1], a[0:3], off"], True),
    (["v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]"], False),
    (["v_mfma_f32_32x32x16_bf16 a[0:15], v[4:7], v[8:11], a[0:15]", "v_mul_f32_e32 v5, v1, v2", "s_cbranch_scc1 65533 <f+0x0>"], True)])
def test_the_check_of_distances(lines, wrong):
    """(The last one's second instruction is followed by the first again.)"""
    text = "\n".join(f"\t{line.split(' <')[0]} // {16 * i:012X}: 00000000 {'<' + line.split(' <')[1] if ' <' in line else ''}" for i, line in enumerate(lines))
    assert bool(violations(parse(text))) == wrong
