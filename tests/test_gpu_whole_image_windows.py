"""Layers whose window is the whole feature map: taken as 1 x 1 windows on vectors where the map is contiguous, as windows where it is a range of a
wider buffer."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import rel_to_range, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("c,h,w,n,batch,kind", [(512, 7, 7, 72, 3, "linear"), (8, 3, 5, 24, 1, "linear"), (40, 6, 6, 48, 17, "conv"),
                                                (24, 1, 9, 16, 2, "conv"), (32, 4, 4, 40, 5, "concat")])
def test_window_is_the_image(c, h, w, n, batch, kind, dt):
    b = graphs._Builder("flat", dt, 100 * c + n, graphs.IN_IMAGE, 8, h, w)
    x = b.conv(-1, c, 1, act=wl.ACT_RELU, bias_std=0.3)
    if kind == "linear":
        x = b.linear(x, n, act=wl.ACT_RELU, bias_std=0.3)
    else:
        if kind == "concat":                     # the first of two concatenations in one buffer: read with the buffer's pitch
            x = b.concat(x, b.conv(x, 16, 1, bias_std=0.3))
            c += 16
        wo, bo = b.normal((n, c, h, w), (2.0 / (c * h * w)) ** 0.5), b.normal((n,), 0.3)
        y = b.add(graphs.Layer(graphs.OP_CONV, x, -2, graphs.KIND_IMAGE, n, 1, 1, h, w, 1, 0, 1, wl.ACT_RELU, w_off=wo, b_off=bo))
        if kind == "concat":
            b.concat(x, b.conv(x, 8, 1, bias_std=0.3))
        x = y
    b.linear(x, 16, std=n ** -0.5)
    m = b.finish()
    x_in = wl.make_input(m, batch)
    got = run_gpu(m, x_in)
    # up to three layers stored in 16 bits before the last one, 2^-9 (2^-12) of a value each: the bound is four of them
    assert np.isfinite(got).all() and rel_to_range(got, orc.run_model(m, x_in)) <= (2.0 ** -7 if dt == wl.DT_BF16 else 2.0 ** -10)
