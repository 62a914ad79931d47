"""Wait states that inline assembly has to keep by itself, in the code built
for gfx950: the assembler takes an asm string as it stands, so a scalar write
of M0 needs one instruction (or s_nop) before an LDS DMA that uses it, and a
scalar register written by the vector unit five before a buffer instruction
that reads it, and one that writes part of a register (SDWA) one before the
vector instruction that reads the register.  Checked on the disassembly of
every kernel of the library, in program order."""
import os
import re
import shutil
import subprocess

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                   "paper_2402_17152_amd", "libhstu.so")
OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
SGPRS = re.compile(r"\bs\[(\d+):(\d+)\]|\bs(\d+)\b")


VGPRS = re.compile(r"\bv\[(\d+):(\d+)\]|\bv(\d+)\b")


def _regs(pattern, text):
    out = set()
    for lo, hi, one in pattern.findall(text):
        out |= {int(one)} if one else set(range(int(lo), int(hi) + 1))
    return out


def faults(lines):
    """Instructions (text) that come too early.  `lines`: a disassembly."""
    bad = []
    m0_age = 99            # wait states since M0 was written by the scalar unit
    valu_age = {}          # the same per scalar register written by the vector unit
    part = set()           # vector registers the instruction before wrote a part of
    for line in lines:
        ins = line.split("//")[0].strip()
        m = re.match(r"([a-z]\w+)\s*(.*)", ins)
        if not m or line[:1] not in "\t ":
            continue
        op, args = m.groups()
        if op.startswith(("buffer_", "global_", "scratch_")):
            if re.search(r"\blds\b|_lds_", ins) and m0_age < 1:
                bad.append(ins)
            if any(valu_age.get(s, 99) < 5 for s in _regs(SGPRS, args)):
                bad.append(ins)
        dst = args.split(",")[0]
        merges = re.search(r"dst_sel:(BYTE|WORD)", ins)
        if op.startswith("v_") and part & _regs(VGPRS, args if merges else args[len(dst):]):
            bad.append(ins)
        part = _regs(VGPRS, dst) if merges else set()
        states = int(args) + 1 if op == "s_nop" else 1
        m0_age += states
        valu_age = {s: a + states for s, a in valu_age.items() if a + states < 5}
        if op.startswith("s_") and dst == "m0":
            m0_age = 0
        if op.startswith("v_"):
            for s in _regs(SGPRS, dst):
                valu_age[s] = 0
    return bad


def test_rules():
    """The rules on listings that break and that keep them."""
    load = "\tbuffer_load_dwordx4 v1, s[8:11], 0 offen lds"
    assert faults(["\ts_mov_b32 m0, s4", load]) == [load.strip()]
    assert faults(["\ts_mov_b32 m0, s4", "\ts_nop 0", load]) == []
    read = "\tv_readfirstlane_b32 s9, v0"
    assert faults([read, "\ts_nop 3", load]) == [load.strip()]
    assert faults([read, "\ts_nop 4", load]) == []
    sdwa = "\tv_sub_u32_sdwa v3, v4, v5 clamp dst_sel:BYTE_%d dst_unused:UNUSED_PRESERVE"
    assert faults([sdwa % 1, sdwa % 2]) == [(sdwa % 2).strip()]
    assert faults([sdwa % 1, "\ts_nop 0", sdwa % 2]) == []


def test_built_kernels(tmp_path):
    if not os.path.exists(LIB) or not os.path.exists(OBJDUMP):
        pytest.skip("needs the built library and llvm-objdump")
    shutil.copy(LIB, tmp_path / "lib.so")
    subprocess.run([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, check=True,
                   stdout=subprocess.DEVNULL)
    codes = sorted(p for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert codes
    dma = 0
    for code in codes:
        text = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", code.name], cwd=tmp_path,
                              check=True, capture_output=True, text=True).stdout
        bad = faults(text.splitlines())
        dma += len(re.findall(r"buffer_load_dword\w* .* lds\b", text))
        assert not bad, f"{len(bad)} too early, first: {bad[0]}"
    assert dma > 100
