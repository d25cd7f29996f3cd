"""Depthwise and pointwise layer in one launch: every shape of the kernel at ragged pixels, channels and steps, against the oracle and against the two
launches."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


def _model(dt, c, n, h, w, stride, pad, act_d, act_p, res):
    b = graphs._Builder("dwpw", dt, c + n + h, graphs.IN_IMAGE, 8, h, w)
    x = b.conv(-1, c, 1, act=wl.ACT_RELU, bias_std=0.3)
    y = b.conv(x, c, 3, stride, pad, act_d, groups=c, bias_std=0.5)
    r = -2
    if res:                                      # the residual of an inverted bottleneck comes from before its expansion
        b = graphs._Builder("dwpw", dt, c + n + h, graphs.IN_IMAGE, 8, h, w)
        r = b.conv(-1, n, 1, bias_std=0.3)
        x = b.conv(r, c, 1, act=wl.ACT_RELU, bias_std=0.3)
        y = b.conv(x, c, 3, stride, pad, act_d, groups=c, bias_std=0.5)
    z = b.conv(y, n, 1, 1, 0, act_p, res=r, bias_std=0.5)
    b.maxpool(z, 1, 1, 0)                        # hands the values through
    return b.finish()


def _both(m, x, plan):
    g = GpuModel(m, max_batch=x.shape[0])
    try:
        os.environ["ECLIP_DWPW"] = plan
        got, (_, n_k, _) = g.run(x, table=[0], timing=True)
        os.environ["ECLIP_DWPW"] = "0,0"
        ref, (_, n_ref, _) = g.run(x, table=[0], timing=True)
    finally:
        os.environ.pop("ECLIP_DWPW", None)
        g.free()
    assert n_ref - n_k == 1
    return got, ref


# one to 30 steps of 32 channels, ragged last ones; pixels below, at and above a tile; channel counts that are no multiple of a column
CASES = [
    (wl.DT_F16, 32, 16, 13, 11, 1, 1, wl.ACT_RELU6, wl.ACT_NONE, False, 2),
    (wl.DT_BF16, 40, 24, 9, 10, 2, 1, wl.ACT_RELU6, wl.ACT_NONE, False, 3),
    (wl.DT_F16, 144, 24, 7, 9, 1, 1, wl.ACT_RELU6, wl.ACT_NONE, True, 1),
    (wl.DT_BF16, 8, 100, 5, 3, 1, 2, wl.ACT_NONE, wl.ACT_RELU, False, 1),
    (wl.DT_BF16, 192, 68, 4, 4, 1, 0, wl.ACT_GELU, wl.ACT_GELU, False, 4),
    (wl.DT_F16, 960, 160, 7, 7, 1, 1, wl.ACT_RELU, wl.ACT_RELU6, True, 1),
]


@pytest.mark.parametrize("tn,wk", [(tn, wk) for tn in (1, 2, 4) for wk in (1, 2, 4, 8)])
def test_shapes(tn, wk):
    for i, (dt, c, n, h, w, stride, pad, act_d, act_p, res, batch) in enumerate(CASES):
        m = _model(dt, c, n, h, w, stride, pad, act_d, act_p, res)
        x = wl.make_input(m, batch)
        got, ref = _both(m, x, f"{tn},{wk}")
        # three layers stored in 16 bits, 2^-9 (2^-12) of a value each, and a residual: the bound is four of them; against the two launches only
        # the order of the sums differs, so that single values round to their neighbour
        tol = 2.0 ** -7 if dt == wl.DT_BF16 else 2.0 ** -10
        assert np.isfinite(got).all(), (i, tn, wk)
        assert rel_to_range(got, orc.run_model(m, x)) <= tol and rel_to_range(got, ref) <= tol, (i, tn, wk)


def test_border_and_lowest_values():
    """Infinities travel through both layers as they do through two launches, and padding stays zero beside them."""
    m = _model(wl.DT_BF16, 32, 16, 6, 7, 1, 1, wl.ACT_NONE, wl.ACT_NONE, False)
    x = wl.make_input(m, 1)
    x[0, :, 0, 0] = 3.0e38
    got, ref = _both(m, x, "1,1")
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and not np.isfinite(got).all()
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= 2.0 ** -6 * np.abs(ref[ok]).max()
