"""The persistent GEMM writes its matrix instructions in inline assembly, which the compiler does not recognise as such: it adds no
wait states around them.  The source keeps a distance by construction (operands come from LDS reads, accumulators are read
behind an s_nop); this checks, in the code of the built library, that the compiler left it so."""
import os
import re
import struct
import subprocess

import pytest

from paper_2509_06040_amd import binding as br

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(path):
    """The gfx950 code objects of a shared library (offload bundles: magic, count, then offset, size and triple of each entry)."""
    blob = open(path, "rb").read()
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in triple:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def regs(operand):
    """Registers of an operand text: v7, v[4:7], a[0:3] -> {(kind, number)}."""
    m = re.fullmatch(r"([va])(?:(\d+)|\[(\d+):(\d+)\])", operand.strip())
    if not m:
        return set()
    lo, hi = (int(m[2]), int(m[2])) if m[2] else (int(m[3]), int(m[4]))
    return {(m[1], i) for i in range(lo, hi + 1)}


def hazards(lines):
    """(matrix instructions, violations).  Distances in wait states: one per instruction, N + 1 for s_nop N.  Needed between a
    vector instruction's write and a matrix instruction's read: 2; between a matrix instruction's write and another reader: at
    most 19 (the longest instructions; those here have 8 passes)."""
    now, count, bad = 0, 0, []
    valu, mfma = {}, {}            # register -> time of its last write
    for line in lines:
        m = re.match(r"\s+([a-z0-9_]+)\s*(.*?)\s*(?://|$)", line)
        if not m:
            continue
        op, args = m[1], [a for a in re.split(r",\s*(?![^\[]*\])", m[2])]
        if op.startswith("v_mfma"):
            count += 1
            for r in set().union(*(regs(a) for a in args[1:4])):
                if now - valu.get(r, -99) <= 2:
                    bad.append(line)
            for r in regs(args[0]):
                mfma[r] = now
                valu.pop(r, None)
        elif op.startswith("v_"):
            for r in set().union(*(regs(a) for a in args[1:]), set()):
                if now - mfma.get(r, -99) <= 19:
                    bad.append(line)
            for r in regs(args[0]):
                valu[r] = now
                mfma.pop(r, None)
        now += int(args[0], 0) + 1 if op == "s_nop" else 1
    return count, bad


def test_the_checker_sees_a_hazard():
    ok = ["\tv_mov_b32_e32 v4, v9", "\ts_nop 1", "\tv_mfma_f32_16x16x32_bf16 a[0:3], v[4:7], v[8:11], a[0:3]", "\ts_nop 15", "\ts_nop 15",
          "\tv_accvgpr_read_b32 v1, a2"]
    assert hazards(ok) == (1, [])
    assert len(hazards(ok[:1] + ok[2:])[1]) == 1           # the operand's write too close
    assert len(hazards(ok[:3] + ok[4:])[1]) == 1           # the result read too soon
    assert len(hazards(["\tv_accvgpr_write_b32 a3, v1"] + ok[2:3])[1]) == 1


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump is missing")
def test_wait_states_around_the_inline_matrix_instructions(tmp_path):
    kernels = 0
    for i, obj in enumerate(code_objects(br.LIB_PATH)):
        if b"gemm_bf16_stream_kernel" not in obj:
            continue
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            name, _, body = part.partition("\n")
            if "gemm_bf16_stream_kernel" not in name:
                continue
            count, bad = hazards(body.split("\n"))
            assert count >= 4 * 8 * 4 * 2 and not bad, (name, count, bad[:5])
            kernels += 1
    assert kernels == 20


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="llvm-objdump is missing")
def test_wait_states_where_outputs_stay_in_the_caches(tmp_path):
    """The same of the kernels that store bf16 outputs plainly (five tile heights, with and without GELU)."""
    kernels = 0
    for i, obj in enumerate(code_objects(br.LIB_PATH)):
        if b"gemm_bf16_stream_keep_kernel" not in obj:
            continue
        f = tmp_path / ("%d.co" % i)
        f.write_bytes(obj)
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(f)], capture_output=True, text=True, check=True).stdout
        for part in re.split(r"\n(?=[0-9a-f]+ <)", text):
            name, _, body = part.partition("\n")
            if "gemm_bf16_stream_keep_kernel" in name:
                count, bad = hazards(body.split("\n"))
                assert count >= 4 * 8 * 4 * 2 and not bad, (name, count, bad[:5])
                kernels += 1
    assert kernels == 10
