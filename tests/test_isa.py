"""Machine-code checks of the bf16 attention kernels, compiled here for gfx950.

The MLA kernel keeps its output accumulators in the AGPR file and updates them
only with MFMAs written as inline assembly; the compiler schedules around
those statements without knowing that they are MFMAs.  A result of such an
MFMA is readable 18 wait states after it issues.  These tests compile the
kernels exactly as the build does and walk the generated assembly:

  * no instruction other than an MFMA reads or writes a register that an
    inline-assembly MFMA wrote until an s_nop sequence of at least 18 wait
    states has passed (the kernels' explicit wait before the epilogue);
  * no accumulator is copied between AGPRs (v_accvgpr_mov), which the
    compiler only does when it moves a value it does not see being written.

  * no vector-memory instruction reads a scalar register within five wait
    states of a VALU instruction writing it (the LDS-DMA loads are inline
    assembly too, and their base address comes through v_readfirstlane).

The walkers are checked on small synthetic listings first."""
import os
import re
import subprocess

import pytest

from paper_2606_17107_amd import build as B

pytestmark = pytest.mark.skipif(not os.path.exists(B.hipcc()), reason="hipcc not available")


def _regs(tok):
    m = re.match(r"^([va])(\d+)$", tok)
    if m:
        return {(m.group(1), int(m.group(2)))}
    m = re.match(r"^([va])\[(\d+):(\d+)\]$", tok)
    if m:
        return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)}
    return set()


def _split(line):
    body = line.split(";")[0].strip()
    parts = body.split(None, 1)
    if not parts:
        return "", []
    if len(parts) == 1:
        return parts[0], []
    return parts[0], [o.strip() for o in re.split(r",(?![^\[]*\])", parts[1])]


def hazards(asm_text):
    """(kernel, line, kind, text) for every violation in an assembly listing."""
    found = []
    starts = [m.start() for m in re.finditer(r"^_ZN\S*kernel\S*:", asm_text, re.M)]
    for s0 in starts:
        name = asm_text[s0:asm_text.index(":", s0)]
        end = asm_text.find(".Lfunc_end", s0)
        lines = asm_text[s0:end if end > 0 else len(asm_text)].split("\n")
        pending, nops, in_asm = set(), 0, False
        for k, line in enumerate(lines):
            if ";;#ASMSTART" in line:
                in_asm = True
                continue
            if ";;#ASMEND" in line:
                in_asm = False
                continue
            op, ops = _split(line)
            if not op or op.endswith(":") or op.startswith(".") or op.startswith(";"):
                continue
            if op == "v_accvgpr_mov_b32":
                found.append((name, k, "AGPR copy", line.strip()))
            if op == "s_nop":
                nops += int(ops[0], 0) + 1
                if nops >= 18:
                    pending.clear()
                continue
            nops = 0
            if op.startswith("v_mfma"):
                srcs = set().union(*(_regs(o) for o in ops[1:3]))
                if srcs & pending:
                    found.append((name, k, "MFMA operand read before the wait", line.strip()))
                if in_asm:
                    pending |= _regs(ops[0])
                else:
                    pending -= _regs(ops[0])
                continue
            regs = set().union(*(_regs(o) for o in ops)) if ops else set()
            if regs & pending:
                found.append((name, k, "result used before the wait", line.strip()))
    return found


def test_walker_flags_early_reads():
    ok = """_ZN3fooL6kernelEv:
	;;#ASMSTART
	v_mfma_f32_32x32x16_bf16 a[0:15], v[0:3], v[4:7], a[0:15]
	;;#ASMEND
	v_add_f32_e32 v8, v9, v10
	;;#ASMSTART
	s_nop 7
	s_nop 7
	s_nop 7
	;;#ASMEND
	v_accvgpr_read_b32 v11, a3
.Lfunc_end0:
"""
    assert hazards(ok) == []
    early = ok.replace("	v_add_f32_e32 v8, v9, v10\n", "	v_accvgpr_read_b32 v8, a2\n")
    assert [h[2] for h in hazards(early)] == ["result used before the wait"]
    copy = ok.replace("	v_add_f32_e32 v8, v9, v10\n", "	v_accvgpr_mov_b32 a40, a2\n")
    assert {h[2] for h in hazards(copy)} == {"AGPR copy", "result used before the wait"}
    # the compiler's own MFMAs are left to the compiler
    builtin = ok.replace(";;#ASMSTART\n	v_mfma", ";\n	v_mfma", 1)
    assert hazards(builtin.replace("	v_add_f32_e32 v8, v9, v10\n", "	v_accvgpr_read_b32 v8, a2\n")) == []


@pytest.mark.parametrize("src", ["attn_mla_bf16.hip", "attn_gqa_bf16.hip"])
def test_attention_kernel_assembly(src, tmp_path):
    path = os.path.join(B.CSRC, src)
    out = tmp_path / (src + ".s")
    cmd = [B.hipcc()] + B.compile_flags() + B.FILE_FLAGS.get(src, []) + [
        "--cuda-device-only", "-S", path, "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    text = out.read_text()
    assert "v_mfma" in text
    found = hazards(text)
    assert not found, found[:10]


def scalar_base_hazards(asm_text):
    """(line, wait states, text) of every vector-memory instruction that reads a scalar register fewer
    than five wait states after a VALU instruction wrote it.  Lines are taken in listing order."""
    found, age = [], {}
    for k, line in enumerate(asm_text.split("\n")):
        op, ops = _split(line)
        if not op or op.endswith(":") or op.startswith((".", ";")):
            continue
        if op.startswith(("global_", "buffer_", "flat_", "scratch_")):
            for o in ops:
                m = re.match(r"^s\[(\d+):(\d+)\]$", o.split()[0]) if o else None
                for r in range(int(m.group(1)), int(m.group(2)) + 1) if m else ():
                    if age.get(r, 99) < 5:
                        found.append((k, age[r], line.strip()))
        step = int(ops[0], 0) + 1 if op == "s_nop" else 1
        age = {r: a + step for r, a in age.items() if a + step < 5}
        dst = ops[0] if ops else ""
        m = re.match(r"^s(?:(\d+)|\[(\d+):(\d+)\])$", dst)
        if m and op.startswith("v_"):
            lo = int(m.group(1) or m.group(2))
            for r in range(lo, int(m.group(3) or lo) + 1):
                age[r] = 0
        elif m:
            lo = int(m.group(1) or m.group(2))
            for r in range(lo, int(m.group(3) or lo) + 1):
                age.pop(r, None)
    return found


def test_walker_flags_early_scalar_reads():
    load = "\tglobal_load_lds_dwordx4 v5, s[4:5]\n"
    assert scalar_base_hazards("\tv_readfirstlane_b32 s4, v2\n\ts_mov_b32 m0, s7\n\ts_nop 0\n" + load)
    assert scalar_base_hazards("\tv_readlane_b32 s5, v254, 34\n\ts_nop 3\n" + load)
    assert not scalar_base_hazards("\tv_readfirstlane_b32 s4, v2\n\ts_nop 4\n" + load)
    assert not scalar_base_hazards("\tv_readfirstlane_b32 s6, v2\n" + load)      # another register
    assert not scalar_base_hazards("\tv_readfirstlane_b32 s4, v2\n\ts_mov_b32 s4, s8\n" + load)


@pytest.mark.parametrize("src", sorted(f for f in os.listdir(B.CSRC) if f.startswith("attn_") and f.endswith(".hip")))
def test_loads_wait_for_their_scalar_base(src, tmp_path):
    out = tmp_path / (src + ".s")
    cmd = [B.hipcc()] + B.compile_flags() + B.FILE_FLAGS.get(src, []) + [
        "--cuda-device-only", "-S", os.path.join(B.CSRC, src), "-o", str(out)]
    subprocess.run(cmd, check=True, capture_output=True)
    text = out.read_text()
    assert "global_load_lds" in text
    found = scalar_base_hazards(text)
    assert not found, found[:10]
