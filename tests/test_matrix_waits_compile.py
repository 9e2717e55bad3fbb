"""The matrix instructions that the GEMM file writes as assembly: the compiler keeps none of the hardware's wait states for them, so
the assembly of every kernel built from the file is read for those that could be missed: a vector instruction that writes an operand
right before its matrix instruction (2 wait states), also over the branch back to a loop's begin; anything but a matrix instruction that
names an accumulator inside the loops, where the last one's result may not be there yet; and a read of one right behind them (16)."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2512_20953_amd import build

MFMA = "v_mfma_f32_16x16x32"


def _registers(text):
    for kind, a, b, one in re.findall(r"\b([va])(?:\[(\d+):(\d+)\]|(\d+))", text):
        for k in range(int(a or one), int(b or one) + 1):
            yield kind, k


def _check(name, body):
    """One kernel's assembly; returns how many branches back it has, or None if it has no such matrix instruction."""
    lines = [l.strip() for l in body.split("\n")]
    lines = [l for l in lines if l and l[0] != ";" and (l[0] != "." or re.match(r"\.L\w+:", l))]
    code = [l for l in lines if l[0] != "."]
    first, n = {}, 0                                      # label -> index in code
    for l in lines:
        if l[0] == ".":
            first[l.split(":")[0]] = n
        else:
            n += 1
    at = [i for i, l in enumerate(code) if l.startswith(MFMA)]
    if not at:
        return None
    # the two instructions before each: in the text, and at a branch back over its target
    runs, backs = [code[max(i - 2, 0):i + 1] for i in at], 0
    for i, l in enumerate(code):
        target = re.match(r"s_c?branch\w* +(\.L\w+)", l)
        if target and first[target.group(1)] <= i:
            backs += 1
            joined = code[max(i - 1, 0):i + 1] + code[first[target.group(1)]:][:2]
            runs += [joined[max(k - 2, 0):k + 1] for k, j in enumerate(joined) if j.startswith(MFMA)]
    for run in runs:
        used = set(_registers(run[-1]))
        for l in run[:-1]:
            if l.startswith("v_") and not l.startswith("v_mfma"):
                assert not used & set(_registers(l.split(",")[0])), (name, l, run[-1])
    accumulators = set().union(*(_registers(code[i].split(",")[0]) for i in at))
    for l in code[at[0]:at[-1] + 1]:
        assert l.startswith(MFMA) or not accumulators & set(_registers(l)), (name, l)
    behind = code[at[-1] + 1:]
    wait = next(i for i, l in enumerate(behind) if l == "s_nop 15")
    assert not any(kind == "a" for l in behind[:wait] for kind, _ in _registers(l)), name
    return backs


@pytest.mark.skipif(not shutil.which("hipcc"), reason="no compiler")
def test_wait_states_around_matrix_instructions(tmp_path):
    asm = tmp_path / "gemm.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm.hip"), "-o", str(asm)], check=True,
                   capture_output=True)
    found = [_check(*m) for m in re.findall(r"^(_ZN2ah\S+):[^\n]*\n(.*?)s_endpgm", asm.read_text(), re.S | re.M)]
    backs = [n for n in found if n is not None]
    assert len(backs) > 40 and all(n > 0 for n in backs)


LOOP = ["s_nop 0", ".LBB0_1:", MFMA + "_bf16 a[0:3], v[8:11], v[4:7], a[0:3]", MFMA + "_bf16 a[4:7], v[8:11], v[12:15], a[4:7]", "s_nop 0", "s_nop 0",
        "s_cbranch_scc1 .LBB0_1", "s_nop 15", "v_accvgpr_read_b32 v0, a0"]


@pytest.mark.parametrize("at,line", [(2, "v_mov_b32_e32 v9, v1"), (4, "v_accvgpr_read_b32 v20, a2"), (3, "v_accvgpr_write_b32 a5, v1"),
                                     (6, "v_add_u32_e32 v8, 4, v8"), (7, "v_accvgpr_read_b32 v20, a6")])
def test_what_is_looked_for_is_found(at, line):
    """A loop as it should be, and the same with one instruction more where it may not stand."""
    assert _check("loop", "\n".join(LOOP)) == 1
    with pytest.raises(AssertionError):
        _check("loop", "\n".join(LOOP[:at] + [line] + LOOP[at:]))
