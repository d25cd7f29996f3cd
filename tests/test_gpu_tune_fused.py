"""eclip_model_tune on layers that requests give a launch together with their neighbours: a convolution is timed with the max-pool behind it, and layers that
another kernel takes are left out."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


@pytest.fixture
def switch():
    kept = {}

    def _switch(name, value):
        kept.setdefault(name, os.environ.get(name))
        os.environ[name] = value
    yield _switch
    for name, value in kept.items():
        os.environ.pop(name) if value is None else os.environ.__setitem__(name, value)


def _pooled(cin, cout, h, w):
    b = graphs._Builder("pooled", wl.DT_BF16, h + w, graphs.IN_IMAGE, cin, h, w)
    x = b.conv(-1, cin, 1, bias_std=0.3)
    x = b.conv(x, cout, 3, 1, 1, wl.ACT_RELU, bias_std=0.5)
    x = b.maxpool(x, 2, 2, 0)
    b.conv(x, 16, 1, bias_std=0.3)
    return b.finish()


def _launches(g, m, batch):
    return g.h.profile_group_served(0, 0, batch, 1)[1]


@pytest.mark.parametrize("cin,cout,h,w,batch", [(64, 128, 112, 112, 4), (64, 128, 111, 113, 4), (64, 64, 27, 30, 2)])
def test_a_convolution_is_timed_with_its_pool(cin, cout, h, w, batch):
    m = _pooled(cin, cout, h, w)
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch)
    try:
        before = _launches(g, m, batch)
        # three convolutions, and the second one once more as the unit that requests launch
        assert g.h.tune(0, batch=batch, iters=3) == 4
        assert g.h.tune(0, batch=batch, iters=1) == 0
        if h > 100:                              # the pool's launch is a quarter of both: it stays in the convolution's
            assert _launches(g, m, batch) == before
        got = g.run(x)
        assert np.array_equal(got, g.run(x))
        if h < 100:
            assert rel_to_range(got, orc.run_model(m, x)) <= 2.0 ** -6       # three roundings to bf16 in a row
    finally:
        g.free()


def test_layers_that_never_share_a_launch_are_timed_alone(switch):
    switch("ECLIP_NO_PAIRS", "1")
    m = _pooled(64, 64, 27, 30)
    g = GpuModel(m, max_batch=2)
    try:
        assert g.h.tune(0, batch=2, iters=1) == 3
    finally:
        g.free()
