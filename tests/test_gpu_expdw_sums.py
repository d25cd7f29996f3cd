"""Expansion, depthwise and pointwise layer in one launch by the library's own choice: the same bits as apart, on sizes of both expansions' plans and all counts of
slices, and apart where the sums would differ."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from gpu_util import GpuModel

pytestmark = pytest.mark.gpu

R6, RELU, NONE, GELU = wl.ACT_RELU6, wl.ACT_RELU, wl.ACT_NONE, wl.ACT_GELU
UNMASKED, CU64, CU128 = 0, 2, 3                  # streams of the shared pool


def _model(dt, h, w, cin, c, n, stride, acts, res):
    b = graphs._Builder("bottleneck", dt, cin + c + n + h, graphs.IN_IMAGE, 8, h, w)
    x = b.conv(-1, cin, 1, bias_std=0.3)
    y = b.conv(x, c, 1, act=acts[0], bias_std=0.5)
    d = b.conv(y, c, 3, stride, 1, acts[1], groups=c, bias_std=0.5)
    b.maxpool(b.conv(d, n, 1, 1, 0, acts[2], res=x if res else -2, bias_std=0.5), 1, 1, 0)       # hands the values through
    return b.finish()


def _both(m, batch, stream):
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch)
    try:
        one, (_, n_one, _) = g.run(x, table=[stream], timing=True)
        os.environ["ECLIP_EXPDW"] = "0"
        two, (_, n_two, _) = g.run(x, table=[stream], timing=True)
    finally:
        os.environ.pop("ECLIP_EXPDW", None)
        g.free()
    return one, two, n_two - n_one


@pytest.mark.parametrize("stream,dt,batch,h,w,cin,c,n,stride,acts,res", [
    (UNMASKED, wl.DT_BF16, 1, 56, 56, 16, 96, 24, 2, (R6, R6, NONE), False), (UNMASKED, wl.DT_F16, 1, 27, 30, 24, 144, 24, 1, (R6, R6, NONE), True),
    (CU64, wl.DT_BF16, 1, 27, 30, 24, 136, 32, 1, (GELU, NONE, RELU), False), (CU64, wl.DT_F16, 2, 25, 23, 24, 136, 32, 2, (NONE, R6, GELU), False),
    (CU64, wl.DT_F16, 3, 28, 28, 32, 192, 32, 1, (R6, R6, NONE), True),         # the expansion on an LDS tile
    (CU64, wl.DT_BF16, 3, 28, 28, 32, 192, 64, 2, (RELU, R6, NONE), False), (CU128, wl.DT_BF16, 8, 56, 56, 24, 144, 24, 1, (R6, R6, NONE), True),
    (CU64, wl.DT_BF16, 1, 20, 20, 32, 64, 32, 1, (R6, R6, NONE), True), (CU64, wl.DT_F16, 1, 20, 20, 32, 32, 32, 1, (R6, R6, NONE), True),         # two slices, one
    (UNMASKED, wl.DT_BF16, 1, 14, 14, 64, 384, 64, 1, (R6, R6, NONE), True), (CU128, wl.DT_F16, 1, 14, 14, 64, 384, 64, 1, (R6, R6, NONE), True),  # two and three
    (CU128, wl.DT_BF16, 1, 15, 13, 48, 256, 64, 1, (GELU, R6, RELU), False), (CU128, wl.DT_BF16, 1, 14, 14, 96, 512, 64, 1, (R6, R6, NONE), False),  # steps of
    (UNMASKED, wl.DT_F16, 2, 14, 13, 72, 264, 40, 1, (R6, NONE, NONE), False),                                                                     # the expansion
])
def test_one_launch_gives_the_same_bits(stream, dt, batch, h, w, cin, c, n, stride, acts, res):
    one, two, fewer = _both(_model(dt, h, w, cin, c, n, stride, acts, res), batch, stream)
    assert fewer == 1                            # the depthwise and the pointwise layer share a launch apart, too
    assert np.isfinite(one).all() and np.array_equal(one, two)


def test_other_sums_stay_apart():
    # 14 x 14 x 64 at batch 3 on 64 CUs: the depthwise + pointwise kernel shares its slices among four wavefronts, the one launch among eight
    one, two, fewer = _both(_model(wl.DT_F16, 14, 14, 64, 384, 64, 1, (R6, R6, NONE), True), 3, CU64)
    assert fewer == 0 and np.array_equal(one, two)
