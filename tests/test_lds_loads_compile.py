"""Loads into LDS as builtin and as assembly in one kernel: both go where M0 points, so the compiler has to set M0 again for a builtin
that follows an assembly statement.  Read from the assembly of a small kernel built here."""
import shutil
import subprocess

import pytest

from paper_2512_20953_amd import build

SOURCE = """
#include "common.h"
namespace ah {
__global__ void probe(const char* a, float* out) {
  __shared__ char lds[4096];
  uint32_t off = threadIdx.x * 16;
  load16_to_lds(a, off, lds);
  load16_to_lds_uncounted(a, off, lds + 1024);
  load16_to_lds(a, off, lds);
  __syncthreads();
  out[threadIdx.x] = ((float*)lds)[threadIdx.x];
}
}
"""


@pytest.mark.skipif(not shutil.which("hipcc"), reason="no compiler")
def test_m0_is_set_again_after_an_assembly_load(tmp_path):
    src, asm = tmp_path / "probe.hip", tmp_path / "probe.s"
    src.write_text(SOURCE)
    subprocess.run(["hipcc", *build.FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)], check=True, capture_output=True)
    seen, m0 = [], None
    for line in asm.read_text().splitlines():
        words = line.replace(",", " ").split()
        if len(words) > 1 and words[0].startswith("s_") and words[1] == "m0":
            m0 = words[2]
        if words and words[0].startswith("global_load_lds"):
            seen.append(m0)
    assert len(seen) == 3 and seen[0] == seen[2] != seen[1], seen
