"""The stated wait for the matrix pipeline ties every accumulator it is given: a
product whose result is no operand of the wait may be scheduled behind it, and its
reader in the next block would then see old values.  The helper is compiled to
compiler IR (gfx950) and the operands of its one statement are counted."""
import os
import re
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

SRC = """
#include "common.h"
using namespace gkv;
__global__ void one(f32x4* x) { f32x4 a = x[0]; mfma_done(a); x[0] = a; }
__global__ void four(f32x4* x) {
  f32x4 a[4] = {x[0], x[1], x[2], x[3]};
  mfma_done(a);
  for (int i = 0; i < 4; ++i) x[i] = a[i];
}
"""


@pytest.mark.skipif(not os.path.exists(HIPCC), reason="hipcc not installed")
def test_every_accumulator_is_an_operand_of_the_wait(tmp_path):
    (tmp_path / "w.hip").write_text(SRC)
    out = tmp_path / "w.ll"
    subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-w", "--offload-device-only", "-emit-llvm", "-S",
                    "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2608_07001_amd", "csrc"),
                    str(tmp_path / "w.hip"), "-o", str(out)], check=True)
    waits = re.findall(r'asm sideeffect "s_nop 15[^"]*", "([^"]*)"', out.read_text())
    assert sorted(w.count("=v") for w in waits) == [1, 4], waits
