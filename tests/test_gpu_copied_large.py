"""The copied tiles whose accumulators fill the accumulation registers (256 x 256, 256 x 192, 192 x 256), through each of their epilogues: storage type
and float outputs with whole groups of eight columns, ragged columns; with a residual and every activation; more than one tile column and row."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import rel_to_range, run_gpu

pytestmark = pytest.mark.gpu


def _model(dt, rows, k, n, act, storage):
    b = graphs._Builder("layers", dt, 31 * n + k + act, graphs.IN_SEQ, k, 1, rows)
    first = b.linear(-1, n - n % 8, std=1.0 / np.sqrt(k), bias_std=0.3)
    out = b.linear(-1, n, act=act, res=first if n % 8 == 0 else -2, std=1.0 / np.sqrt(k), bias_std=0.5)
    if storage:
        b.eltwise(out)                       # passes the rounded values on as floats
    return b.finish()


@pytest.mark.parametrize("tile", [17, 24, 25])
@pytest.mark.parametrize("dt,act,rows,k,n,storage", [
    (wl.DT_BF16, wl.ACT_GELU, 300, 96, 520, True), (wl.DT_F16, wl.ACT_RELU6, 256, 352, 512, True), (wl.DT_F16, wl.ACT_GELU, 257, 72, 264, True),
    (wl.DT_BF16, wl.ACT_GELU, 300, 96, 520, False), (wl.DT_F16, wl.ACT_RELU, 513, 160, 256, False), (wl.DT_BF16, wl.ACT_NONE, 17, 40, 776, False),
    (wl.DT_BF16, wl.ACT_RELU6, 270, 64, 516, False), (wl.DT_F16, wl.ACT_GELU, 270, 64, 515, False),
])
def test_epilogues(tile, dt, act, rows, k, n, storage):
    # Float outputs differ from the oracle by the order of at most 352 additions (2e-4 of the range as for every linear layer here) and by the
    # residual's one rounding, at most 2^-9 (2^-12) of the larger of the two summands; storage outputs are rounded once more.  Twice that is the bound.
    step = 2.0 ** -9 if dt == wl.DT_BF16 else 2.0 ** -12
    tol = 2 * step * (storage + (n % 8 == 0)) + 2e-4
    m = _model(dt, rows, k, n, act, storage)
    x = wl.make_input(m, 1)
    os.environ["ECLIP_GEMM_FORCE"] = f"0,{tile},1"
    try:
        got = run_gpu(m, x)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
    assert np.isfinite(got).all()
    assert rel_to_range(got, orc.run_model(m, x)) <= tol
