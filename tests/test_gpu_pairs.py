"""Two independent layers in one launch of the lean wave-split-K kernel: ragged rows and channels, equal and unlike address forms, outputs of their
own and side by side in one tensor."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


def _model(dt, first, second, joined):
    b = graphs._Builder("pair", dt, 77, graphs.IN_IMAGE, 64, 13, 11)
    x = b.conv(-1, 96, 3, 1, 1, act=wl.ACT_RELU, bias_std=0.3)
    a = b.conv(x, 72, *first, bias_std=0.5)
    c = b.conv(x, 40 if joined else 72, *second, act=wl.ACT_RELU, bias_std=0.5)
    if joined:
        b.concat(a, c)
    else:
        b.eltwise(a, res=c)
    return b.finish()


@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("joined", [False, True])
@pytest.mark.parametrize("first,second", [                     # kernel size, stride, padding
    ((1, 1, 0), (3, 1, 1)), ((3, 1, 1), (1, 1, 0)),            # rows next to a window: both run as windows
    ((1, 2, 0), (3, 2, 1)), ((5, 2, 2), (3, 2, 1)),            # two windows
    ((1, 1, 0), (1, 1, 0)),                                    # two of rows
])
@pytest.mark.parametrize("batch", [1, 3])
def test_two_layers_in_one_launch(dt, joined, first, second, batch):
    m = _model(dt, first, second, joined)
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch)
    try:
        got, t = g.run(x, timing=True)
        os.environ["ECLIP_NO_PAIRS"] = "1"
        try:
            apart, t2 = g.run(x, timing=True)
        finally:
            del os.environ["ECLIP_NO_PAIRS"]
    finally:
        g.free()
    assert t[1] == t2[1] - 1                                   # n_kernels
    exp = orc.run_model(m, x)
    # three roundings to the storage type on the way, at most 2^-9 (2^-12) of a value each; twice that is the bound
    tol = 6 * (2.0 ** -9 if dt == wl.DT_BF16 else 2.0 ** -12)
    assert rel_to_range(got, exp) <= tol and rel_to_range(apart, exp) <= tol
    # against the same layers one launch each only the order of the sums differs: one more rounding, where it falls the other way
    assert np.abs(got - apart).max() <= tol / 3 * np.abs(exp).max()
