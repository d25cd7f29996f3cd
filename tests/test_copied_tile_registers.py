"""Copied tiles whose accumulators the compiler would have to move between the register files gave wrong sums: they are not compiled.  Asked of the compiler."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_12598_amd", "csrc")
pytestmark = pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")

PROGRAM = """
#include "gemm_dma.h"
using namespace eclip;
template __global__ void eclip::conv_gemm_dma_kernel<bf16_t, {bm}, {bn}, 32, 2, 2, {stages}, A_MATRIX>(const uint16_t *, const uint16_t *, unsigned, int, int, int,
    int, int, unsigned, unsigned, unsigned, unsigned, GemmDev, SeDeal);
"""


@pytest.mark.parametrize("bm,bn,stages,fits", [
    (128, 256, 3, True), (192, 256, 5, True), (256, 256, 4, True),    # 128 registers; 192 and 256 with a compute unit to themselves
    (192, 192, 3, False), (192, 192, 6, True),                        # 144 where two workgroups share one; alone by its larger ring
])
def test_accumulators_fit_their_registers(tmp_path, bm, bn, stages, fits):
    src = tmp_path / "tile.hip"
    src.write_text(PROGRAM.format(bm=bm, bn=bn, stages=stages))
    got = subprocess.run(["hipcc", "-x", "hip", "--offload-host-only", "-fsyntax-only", "-std=c++17", "-I", CSRC, "-I", os.path.join(ROOT, "include"), str(src)],
                         capture_output=True, text=True)
    assert (got.returncode == 0) == fits, got.stderr
    assert fits or "accumulators fit the accumulation registers" in got.stderr
