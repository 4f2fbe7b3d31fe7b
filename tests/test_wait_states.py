"""Host-side check of what the assembler is given around inline assembly, into which the compiler's own insertion of
wait states does not look.  A copy into LDS reads its address from M0 and needs one instruction (or s_nop 0) between
the scalar write of M0 and itself; a memory instruction needs five between a vector instruction's write of a scalar
register (a spilled one read back from a lane, say) and its use of it.  Reads the assembly of the library's own
sources; no GPU needed."""
import re
import subprocess

import pytest

from paper_2509_22323_amd import build

INSTRUCTION = re.compile(r"^\s+([a-z][a-z0-9_]+)\b(.*)$")


def instructions(asm):
    for line in asm.splitlines():
        m = INSTRUCTION.match(line.split(";")[0].split("//")[0])
        if m and not m.group(1).startswith("."):
            yield m.group(1), m.group(2)


def copies_too_early(asm):
    """(copies into LDS, those right behind a scalar write of M0)"""
    copies = early = 0
    fresh = False                                          # the instruction before wrote M0
    for op, args in instructions(asm):
        to_lds = "_load_lds_" in op or (op.startswith("buffer_load_") and re.search(r"\blds\b", args) is not None)
        copies += to_lds
        early += to_lds and fresh
        fresh = op.startswith("s_") and re.match(r"\s*m0\b", args) is not None
    return copies, early


def scalars(text):
    """scalar registers named in an instruction's operands"""
    out = {int(n) for n in re.findall(r"\bs(\d+)\b", text)}
    for a, b in re.findall(r"\bs\[(\d+):(\d+)\]", text):
        out |= set(range(int(a), int(b) + 1))
    return out


def scalars_too_early(asm):
    """memory instructions within five wait states of a vector instruction that wrote one of their scalar registers"""
    early, last = 0, []                                    # last: (registers written, wait states it takes) of the newest instructions
    for op, args in instructions(asm):
        if op.startswith(("buffer_", "global_", "flat_", "scratch_")):
            distance = 0
            for written, states in reversed(last):
                early += distance < 5 and bool(written & scalars(args))
                distance += states
        written = scalars(args.split(",")[0]) if op.startswith("v_") else set()
        last = (last + [(written, 1 + int(args) if op == "s_nop" else 1)])[-5:]
    return early


def test_the_check_itself():
    good = "\ts_mov_b32 m0, s3\n\ts_nop 0\n\tbuffer_load_dwordx4 v1, s[0:3], 0 offen lds\n"
    assert copies_too_early(good) == (1, 0)
    assert copies_too_early(good.replace("\ts_nop 0\n", "\t;;#ASMEND\n")) == (1, 1)
    assert copies_too_early("\ts_mov_b32 m0, s3\n\tglobal_load_lds_dwordx4 v1, s[0:1]\n") == (1, 1)
    assert copies_too_early("\ts_mov_b32 m0, s3\n\tbuffer_load_dwordx4 v[0:3], v1, s[0:3], 0 offen\n") == (0, 0)
    use = "\tglobal_load_dwordx4 v[0:3], v4, s[2:3]\n"
    assert scalars_too_early("\tv_readlane_b32 s3, v9, 0\n" + "\ts_nop 3\n" + use) == 1
    assert scalars_too_early("\tv_readlane_b32 s3, v9, 0\n" + "\ts_nop 4\n" + use) == 0
    assert scalars_too_early("\tv_readlane_b32 s4, v9, 0\n" + use) == 0


@pytest.mark.parametrize("source", build.SOURCES)
def test_no_instruction_comes_too_early(source, tmp_path):
    out = tmp_path / "x.s"
    flags = [f for f in build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([build.HIPCC] + flags + ["--offload-device-only", "-S", "-o", str(out), source], capture_output=True, check=True)
    asm = out.read_text()
    copies, early = copies_too_early(asm)
    assert early == 0, f"{early} of {copies} copies"
    assert scalars_too_early(asm) == 0
    assert copies >= 100 or "rapid_attn" not in source     # (the attention kernels are full of them)
