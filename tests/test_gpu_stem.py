"""The kernel of the first layer: windows up to 4 x 4 and 7 x 8, both strides, 1 to 4 planes, ragged tiles and channel counts, with and without the pool."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


def _model(dt, cin, cout, h, w, kh, kw, stride, pad, act, pool, keeps_nan=False):
    b = graphs._Builder("stem", dt, cin * 100 + cout + h, graphs.IN_IMAGE, cin, h, w)
    ho, wo = (h + 2 * pad - kh) // stride + 1, (w + 2 * pad - kw) // stride + 1
    wt, bias = b.normal((cout, cin, kh, kw), (2.0 / (cin * kh * kw)) ** 0.5), b.normal((cout,), 0.5)
    x = b.add(graphs.Layer(graphs.OP_CONV, -1, -2, graphs.KIND_IMAGE, cout, ho, wo, kh, kw, stride, pad, 1, act, w_off=wt, b_off=bias))
    if pool:
        x = b.maxpool(x, 3, 2, 1)
    if keeps_nan:
        b.eltwise(x)                             # hands the values through, NaN too
    else:
        b.maxpool(x, 1, 1, 0)                    # hands the values through
    return b.finish()


@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("cin,cout,h,w,kh,kw,stride,pad,act,batch,pool", [
    (3, 64, 67, 71, 7, 7, 2, 3, wl.ACT_RELU, 2, True),           # 17 x 18 pooled: ragged tiles of both sizes, the pool's window beyond every edge
    (3, 64, 224, 224, 7, 7, 2, 3, wl.ACT_RELU, 3, True),         # more large tiles than compute units
    (4, 40, 70, 66, 3, 4, 2, 1, wl.ACT_NONE, 1, True),           # negative values in the pool; 40 of 64 channels
    (1, 24, 133, 130, 3, 3, 2, 1, wl.ACT_RELU6, 1, True),        # one plane, 24 of 32 channels
    (3, 64, 9, 12, 7, 7, 2, 3, wl.ACT_NONE, 3, True),            # a pooled map of 3 x 3, less than a tile
    (2, 8, 33, 35, 5, 6, 2, 0, wl.ACT_GELU, 3, False),           # 5 x 6 in the 7 x 8 form, no padding
    (3, 64, 37, 45, 3, 3, 1, 1, wl.ACT_RELU, 2, False),          # stride 1: pairs of pixels not aligned
    (3, 32, 9, 5, 4, 3, 1, 2, wl.ACT_NONE, 1, False),            # a map smaller than a tile
    (3, 64, 300, 260, 3, 3, 1, 1, wl.ACT_RELU, 1, False),        # large tiles, ragged on both sides
])
def test_first_layer(cin, cout, h, w, kh, kw, stride, pad, act, batch, pool, dt):
    m = _model(dt, cin, cout, h, w, kh, kw, stride, pad, act, pool)
    x = wl.make_input(m, batch)
    exp = orc.run_model(m, x)
    g = GpuModel(m, max_batch=batch)
    try:
        got, (_, n_k, _) = g.run(x, table=[0], timing=True)
        os.environ["ECLIP_NO_PAIRS"] = "1"
        try:
            ref, (_, n_ref, _) = g.run(x, table=[0], timing=True)
        finally:
            del os.environ["ECLIP_NO_PAIRS"]
    finally:
        g.free()
    assert n_ref - n_k == (2 if pool else 1)
    # one rounding to the storage type, 2^-9 (2^-12) of a value: the bound is twice that.  Two kernels that add in another order may round to
    # neighbouring values, which lie up to 2^-7 (2^-10) of a value apart.
    tol = 2.0 ** -8 if dt == wl.DT_BF16 else 2.0 ** -11
    assert np.isfinite(got).all() and rel_to_range(got, exp) <= tol and rel_to_range(got, ref) <= 2 * tol


def _reach(bad, k, stride, pad):
    """Positions of a map whose window holds a marked one: [H][W] -> [Ho][Wo]."""
    h, w = bad.shape
    kh, kw = k
    ho, wo = (h + 2 * pad - kh) // stride + 1, (w + 2 * pad - kw) // stride + 1
    out = np.zeros((ho, wo), bool)
    padded = np.pad(bad, pad)
    for i in range(ho):
        for j in range(wo):
            out[i, j] = padded[i * stride:i * stride + kh, j * stride:j * stride + kw].any()
    return out


# every window that the kernel pads, in rows, in columns and in both, and one that it does not; with the pool and without, every activation
@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("cin,cout,h,w,kh,kw,stride,pad,act,pool", [
    (3, 64, 70, 71, 7, 7, 2, 3, wl.ACT_NONE, True),
    (3, 64, 70, 71, 7, 7, 2, 3, wl.ACT_RELU, True),
    (3, 32, 41, 38, 7, 7, 2, 3, wl.ACT_RELU6, False),
    (1, 24, 40, 43, 3, 3, 2, 1, wl.ACT_NONE, False),
    (3, 40, 72, 70, 3, 3, 2, 1, wl.ACT_GELU, True),
    (4, 64, 37, 34, 3, 3, 1, 1, wl.ACT_RELU, False),
    (2, 8, 33, 35, 5, 6, 2, 0, wl.ACT_NONE, False),
    (2, 16, 39, 30, 2, 5, 2, 2, wl.ACT_NONE, False),
    (3, 16, 39, 31, 4, 3, 1, 2, wl.ACT_NONE, False),
    (2, 24, 38, 35, 3, 4, 2, 1, wl.ACT_RELU, False),
    (2, 24, 38, 35, 7, 8, 2, 3, wl.ACT_NONE, False),
])
def test_values_that_are_not_finite_stay_in_their_windows(cin, cout, h, w, kh, kw, stride, pad, act, pool, dt):
    m = _model(dt, cin, cout, h, w, kh, kw, stride, pad, act, pool, keeps_nan=True)
    # single pixels at all four parities, then blocks over opposite corners, where whole windows of the pool are NaN
    corner = [(i, j) for i in range(11) for j in range(11)]
    marks = [(np.inf, [(12, 12)]), (np.nan, [(13, 16)]), (-np.inf, [(16, 13)]), (np.inf, [(15, 11), (h - 2, w - 1)]),
             (np.nan, corner + [(h - 1 - i, w - 1 - j) for i, j in corner])]
    clean = np.array(wl.make_input(m, len(marks)))
    x = clean.copy()
    hit = np.zeros((len(marks), h, w), bool)
    for n, (v, at) in enumerate(marks):
        for i, j in at:
            hit[n, i, j] = True
            x[n, n % cin, i, j] = v
    exp = orc.run_model(m, clean)
    reach = np.stack([_reach(a, (kh, kw), stride, pad) for a in hit])
    if pool:
        reach = np.stack([_reach(a, (3, 3), 2, 1) for a in reach])
    away = np.broadcast_to(~reach[:, None], exp.shape)
    g = GpuModel(m, max_batch=len(marks))
    try:
        got = g.run(x, table=[0])
        os.environ["ECLIP_NO_PAIRS"] = "1"
        try:
            ref = g.run(x, table=[0])
        finally:
            del os.environ["ECLIP_NO_PAIRS"]
    finally:
        g.free()
    tol = 2.0 ** -8 if dt == wl.DT_BF16 else 2.0 ** -11          # one rounding to the storage type, twice, as above
    span = float(exp.max() - exp.min())
    assert away.any() and reach.any()
    assert np.isfinite(got[away]).all() and np.abs(got[away] - exp[away]).max() <= tol * span
    # within reach: the values of the separate launches, infinities of the same sign and NaN where these have one
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(got[np.isinf(got)], ref[np.isinf(ref)])
    ok = np.isfinite(ref)
    assert np.abs(got[ok] - ref[ok]).max() <= 2 * tol * span
