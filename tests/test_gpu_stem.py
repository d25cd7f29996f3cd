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


def _model(dt, cin, cout, h, w, kh, kw, stride, pad, act, pool):
    b = graphs._Builder("stem", dt, cin * 100 + cout + h, graphs.IN_IMAGE, cin, h, w)
    ho, wo = (h + 2 * pad - kh) // stride + 1, (w + 2 * pad - kw) // stride + 1
    wt, bias = b.normal((cout, cin, kh, kw), (2.0 / (cin * kh * kw)) ** 0.5), b.normal((cout,), 0.5)
    x = b.add(graphs.Layer(graphs.OP_CONV, -1, -2, graphs.KIND_IMAGE, cout, ho, wo, kh, kw, stride, pad, 1, act, w_off=wt, b_off=bias))
    if pool:
        x = b.maxpool(x, 3, 2, 1)
    b.maxpool(x, 1, 1, 0)                        # hands the values through
    return b.finish()


@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("cin,cout,h,w,kh,kw,stride,pad,act,batch,pool", [
    (3, 64, 67, 71, 7, 7, 2, 3, wl.ACT_RELU, 2, True),           # 17 x 18 pooled: ragged tiles of both sizes, the pool's window beyond every edge
    (3, 64, 224, 224, 7, 7, 2, 3, wl.ACT_RELU, 3, True),         # more large tiles than compute units
    (4, 40, 70, 66, 3, 4, 2, 1, wl.ACT_NONE, 1, True),           # negative values in the pool; 40 of 64 channels
    (1, 24, 133, 130, 3, 3, 2, 1, wl.ACT_RELU6, 1, True),        # one plane, 24 of 32 channels
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
