"""Tiles of the lean wave-split-K kernel dealt to the XCDs in ranges: counts that are no multiple of 8, down the columns and along the rows, one layer and
two per launch."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,n", [(16, 256), (17, 304), (100, 144), (250, 16), (270, 36), (145, 160), (300, 28)])     # tiles of 16 x 16: 16 to 100
@pytest.mark.parametrize("variant,nw", [(3, 4), (4, 8), (5, 16), (0, 4)])
def test_ranges_of_tiles(rows, n, variant, nw):
    m = wl.single_layer("linear", wl.DT_F16, seed=rows + n, rows=rows, k=96, n=n, act=wl.ACT_RELU, bias_std=0.3, std=0.1)
    x = wl.make_input(m, 1)
    os.environ["ECLIP_GEMM_FORCE"] = f"1,{variant},{nw}"
    try:
        got = run_gpu(m, x)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
    # float32 results: every tile written once, sums of 96 products
    assert np.isfinite(got).all() and rel_to_range(got, orc.run_model(m, x)) <= 2e-4


@pytest.mark.parametrize("h,w,c0,c1", [(9, 9, 88, 72), (20, 13, 40, 136), (7, 5, 264, 200)])
def test_two_layers_of_one_launch(h, w, c0, c1):
    b = graphs._Builder("two", wl.DT_BF16, h * w, graphs.IN_IMAGE, 64, h, w)
    x = b.eltwise(-1)
    p = b.conv(x, c0, 1, act=wl.ACT_RELU, bias_std=0.3)
    q = b.conv(x, c1, 3, 1, 1, wl.ACT_RELU, bias_std=0.3)
    b.linear(b.gap(b.concat(p, q)), 24, std=0.1)
    m = b.finish()
    x_in = wl.make_input(m, 2)
    g = GpuModel(m, max_batch=2)
    try:
        got, t = g.run(x_in, timing=True)
        os.environ["ECLIP_NO_PAIRS"] = "1"
        try:
            ref, t2 = g.run(x_in, timing=True)
        finally:
            del os.environ["ECLIP_NO_PAIRS"]
    finally:
        g.free()
    assert t[1] < t2[1]
    exp = orc.run_model(m, x_in)
    # two layers stored in bf16, 2^-9 of a value each, then averaged: the bound is four of them
    assert rel_to_range(got, exp) <= 2.0 ** -7 and rel_to_range(ref, exp) <= 2.0 ** -7
