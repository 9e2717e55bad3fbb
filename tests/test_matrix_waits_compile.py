"""The matrix instructions that the GEMM file writes as assembly: the compiler keeps none of the hardware's wait states for them, so
the assembly of every kernel built from the file is read for the two that could be missed: a vector instruction that writes an operand
right before its matrix instruction (2 wait states), and a read of an accumulator right behind the loop (16)."""
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


@pytest.mark.skipif(not shutil.which("hipcc"), reason="no compiler")
def test_wait_states_around_matrix_instructions(tmp_path):
    asm = tmp_path / "gemm.s"
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", os.path.join(build.CSRC, "gemm.hip"), "-o", str(asm)], check=True,
                   capture_output=True)
    kernels = 0
    for name, body in re.findall(r"^(_ZN2ah\S+):[^\n]*\n(.*?)s_endpgm", asm.read_text(), re.S | re.M):
        lines = [l.strip() for l in body.split("\n")]
        lines = [l for l in lines if l and l[0] not in ";."]
        at = [i for i, l in enumerate(lines) if l.startswith(MFMA)]
        if not at:
            continue
        kernels += 1
        for i in at:
            used = set(_registers(lines[i]))
            for l in lines[max(i - 2, 0):i]:
                if l.startswith("v_") and not l.startswith("v_mfma"):
                    assert not used & set(_registers(l.split(",")[0])), (name, l, lines[i])
        behind = lines[at[-1] + 1:]
        wait = next(i for i, l in enumerate(behind) if l == "s_nop 15")
        assert not any(kind == "a" for l in behind[:wait] for kind, _ in _registers(l)), name
    assert kernels > 40
