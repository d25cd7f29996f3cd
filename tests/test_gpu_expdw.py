"""Pointwise expansion, depthwise 3 x 3 and pointwise layer in one launch: every shape of the kernel at ragged images, channels and slices, against the oracle
and against the launches it replaces."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


def _model(dt, cin, c, n, h, w, stride, acts, res, second_reader=False):
    b = graphs._Builder("bottleneck", dt, cin + c + n + h, graphs.IN_IMAGE, 8, h, w)
    x = b.conv(-1, cin, 1, bias_std=0.3)
    y = b.conv(x, c, 1, act=acts[0], bias_std=0.5)
    d = b.conv(y, c, 3, stride, 1, acts[1], groups=c, bias_std=0.5)
    z = b.conv(d, n, 1, 1, 0, acts[2], res=x if res else -2, bias_std=0.5)
    if second_reader:
        z = b.conv(y, n, 1, stride, 0, res=z)
    b.maxpool(z, 1, 1, 0)                        # hands the values through
    return b.finish()


def _both(m, x, fewer=2):
    g = GpuModel(m, max_batch=x.shape[0])
    try:
        os.environ["ECLIP_EXPDW"] = "1"
        got, (_, n_k, _) = g.run(x, table=[0], timing=True)
        os.environ["ECLIP_EXPDW"], os.environ["ECLIP_DWPW"] = "0", "0,0"
        ref, (_, n_ref, _) = g.run(x, table=[0], timing=True)
    finally:
        os.environ.pop("ECLIP_EXPDW", None)
        os.environ.pop("ECLIP_DWPW", None)
        g.free()
    assert n_ref - n_k == fewer
    return got, ref


R6, NONE = wl.ACT_RELU6, wl.ACT_NONE


@pytest.mark.parametrize("stride", [1, 2])
@pytest.mark.parametrize("dt,cin,c,n,h,w,acts,res,batch", [
    (wl.DT_F16, 16, 96, 24, 13, 11, (R6, R6, NONE), False, 2), (wl.DT_BF16, 24, 144, 24, 9, 10, (R6, R6, NONE), True, 3),
    (wl.DT_F16, 32, 200, 68, 8, 8, (wl.ACT_RELU, NONE, wl.ACT_GELU), False, 1), (wl.DT_BF16, 40, 40, 100, 5, 3, (NONE, R6, R6), False, 2),
    (wl.DT_F16, 64, 384, 64, 7, 6, (R6, R6, NONE), True, 2), (wl.DT_BF16, 96, 576, 160, 4, 4, (wl.ACT_GELU, R6, NONE), False, 1),
    (wl.DT_F16, 88, 960, 320, 7, 7, (R6, R6, NONE), False, 3), (wl.DT_BF16, 72, 24, 12, 1, 2, (R6, NONE, wl.ACT_RELU), False, 1),
])
def test_shapes(stride, dt, cin, c, n, h, w, acts, res, batch):
    m = _model(dt, cin, c, n, h, w, stride, acts, res and stride == 1 and cin == n)
    x = wl.make_input(m, batch)
    got, ref = _both(m, x)
    # four layers stored in 16 bits, 2^-9 (2^-12) of a value each, and a residual: the bound is four of them; against the launches apart only
    # the order of the sums differs, so that single values round to their neighbour
    tol = 2.0 ** -7 if dt == wl.DT_BF16 else 2.0 ** -10
    assert np.isfinite(got).all()
    assert rel_to_range(got, orc.run_model(m, x)) <= tol and rel_to_range(got, ref) <= tol


def test_padding_is_zero_and_infinities_travel():
    # an expansion with a bias and no activation: outside the image stands zero, not the bias; values beyond the type's range become infinite in both forms
    m = _model(wl.DT_BF16, 16, 32, 16, 6, 7, 1, (NONE, NONE, NONE), False)
    x = wl.make_input(m, 1)
    got, ref = _both(m, x)
    assert rel_to_range(got, ref) <= 2.0 ** -7
    x[0, :, 0, 0] = 3.0e38
    got, ref = _both(m, x)
    assert np.array_equal(np.isfinite(got), np.isfinite(ref)) and not np.isfinite(got).all()
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= 2.0 ** -6 * np.abs(ref[ok]).max()


def test_an_expansion_that_others_read_stays_apart():
    m = _model(wl.DT_F16, 32, 64, 32, 8, 8, 1, (R6, R6, NONE), False, second_reader=True)
    x = wl.make_input(m, 2)
    got, ref = _both(m, x, fewer=1)              # depthwise + pointwise still share a launch
    assert rel_to_range(got, ref) <= 2.0 ** -10


def test_an_expansion_of_many_channels_stays_apart():
    m = _model(wl.DT_F16, 104, 128, 32, 6, 6, 1, (R6, R6, NONE), False)
    x = wl.make_input(m, 2)
    got, ref = _both(m, x, fewer=1)
    assert rel_to_range(got, ref) <= 2.0 ** -10


@pytest.mark.parametrize("dt,cin,c,n,stride", [(wl.DT_BF16, 16, 40, 16, 1), (wl.DT_F16, 32, 72, 24, 2), (wl.DT_BF16, 72, 264, 40, 1)])
def test_infinities_stay_out_of_the_channels_that_fill_a_slice(dt, cin, c, n, stride):
    # hidden channels that do not fill their last slice of 32: what stands there for the missing ones must not turn an infinity into a NaN.  All weights are
    # positive, so that the windows that reach the infinite pixel sum to infinity and the others stay finite.
    m = _model(dt, cin, c, n, 9, 8, stride, (NONE, NONE, NONE), False)
    m.weights[:] = np.abs(m.weights)
    x = np.abs(wl.make_input(m, 2))
    x[1, 3, 4, 4] = np.inf
    got, ref = _both(m, x)
    assert np.isposinf(ref).any() and not np.isnan(ref).any() and np.isfinite(ref).any()
    assert np.array_equal(np.isposinf(got), np.isposinf(ref)) and not np.isnan(got).any()
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= (2.0 ** -7 if dt == wl.DT_BF16 else 2.0 ** -10) * np.abs(ref[ok]).max()
