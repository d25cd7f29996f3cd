"""The lean form of the wave-split-K kernel: every tile shape and wavefront count, forced in turn, in its three address forms, where each can
go wrong: slices longer than the steps in flight and wavefronts without a step, ragged rows, channels and K, windows of 1 to 31 taps."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import rel_to_range, run_gpu

pytestmark = pytest.mark.gpu

# Sequence outputs are float32: sums of at most 3000 products associate differently, 2e-4 of the range as for every linear layer here.  Image
# outputs are rounded to the storage type once (2^-9 of a value in bf16, 2^-12 in fp16; twice with a computed residual): the bounds are twice that.
CASES = [
    # 1 x 1, stride 1
    (dict(op="linear", dtype=wl.DT_BF16, rows=33, k=32, n=20, act=wl.ACT_RELU, bias_std=0.3, std=0.2), 1, 2e-4),        # one step, N = 20
    (dict(op="linear", dtype=wl.DT_F16, rows=49, k=3008, n=72, act=wl.ACT_GELU, bias_std=0.3, std=0.02), 1, 3e-4),      # 94 steps
    (dict(op="linear", dtype=wl.DT_BF16, rows=40, k=192, n=192, bias_std=0.3, std=0.1, residual=True), 2, 2e-4),
    # K not a multiple of 32
    (dict(op="linear", dtype=wl.DT_F16, rows=17, k=8, n=12, bias_std=0.3, std=0.3), 1, 2e-4),
    (dict(op="linear", dtype=wl.DT_BF16, rows=70, k=1048, n=68, act=wl.ACT_RELU6, bias_std=2.0, std=0.1), 1, 2e-4),
    (dict(op="conv", dtype=wl.DT_F16, cin=24, cout=144, h=9, w=7, k=1, bias_std=0.5), 3, 2.0 ** -11),
    # windows: 1 x 1 at stride 2, borders on all sides, 25 taps, several images per tile
    (dict(op="conv", dtype=wl.DT_BF16, cin=96, cout=72, h=19, w=17, k=1, stride=2, act=wl.ACT_RELU, bias_std=0.5), 2, 2.0 ** -8),
    (dict(op="conv", dtype=wl.DT_BF16, cin=64, cout=44, h=7, w=5, k=3, stride=1, pad=1, bias_std=0.5, residual=True), 3, 2.0 ** -7),
    (dict(op="conv", dtype=wl.DT_F16, cin=32, cout=40, h=9, w=11, k=5, stride=2, pad=2, act=wl.ACT_RELU, bias_std=0.5), 2, 2.0 ** -11),
    (dict(op="conv", dtype=wl.DT_BF16, cin=160, cout=32, h=6, w=6, k=3, stride=1, pad=2, act=wl.ACT_RELU6, bias_std=0.5), 2, 2.0 ** -8),
]


@pytest.mark.parametrize("variant,nw", [(v, nw) for v in range(6) for nw in (4, 8, 16) if (v, nw) != (2, 16)])
def test_tile(variant, nw):
    os.environ["ECLIP_GEMM_FORCE"] = f"1,{variant},{nw}"
    try:
        for i, (kw, batch, tol) in enumerate(CASES):
            kw = dict(kw)
            m = wl.single_layer(kw.pop("op"), kw.pop("dtype"), seed=300 + i, **kw)
            x = wl.make_input(m, batch)
            got = run_gpu(m, x)
            assert np.isfinite(got).all(), (i, kw)
            assert rel_to_range(got, orc.run_model(m, x)) <= tol, (i, kw)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)


@pytest.mark.parametrize("kh,kw,stride,pad", [(5, 6, 1, 4), (6, 5, 2, 3), (1, 31, 1, 15), (31, 1, 1, 16), (2, 13, 2, 7)])
@pytest.mark.parametrize("variant,nw", [(1, 4), (3, 16), (5, 8)])
def test_windows_of_26_to_31_taps(kh, kw, stride, pad, variant, nw):
    # every tap's bit of the border mask is set for some row and clear for another
    b = graphs._Builder("wide", wl.DT_F16, kh * kw, graphs.IN_IMAGE, 32, 9, 10)
    fan_in = 32 * kh * kw
    w, bias = b.normal((40, 32, kh, kw), (2.0 / fan_in) ** 0.5), b.normal((40,), 0.5)
    h, wd = (9 + 2 * pad - kh) // stride + 1, (10 + 2 * pad - kw) // stride + 1
    b.add(graphs.Layer(graphs.OP_CONV, -1, -2, graphs.KIND_IMAGE, 40, h, wd, kh, kw, stride, pad, 1, wl.ACT_RELU, w_off=w, b_off=bias))
    m = b.finish()
    x = wl.make_input(m, 2)
    os.environ["ECLIP_GEMM_FORCE"] = f"1,{variant},{nw}"
    try:
        got = run_gpu(m, x)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
    assert np.isfinite(got).all()
    assert rel_to_range(got, orc.run_model(m, x)) <= 2.0 ** -11


@pytest.mark.parametrize("k", [72, 96])
def test_an_infinite_row_stays_in_its_row(k):
    # lanes beyond K, rows beyond M and steps beyond a wavefront's slice must not bring another row's values into a sum
    m = wl.single_layer("linear", wl.DT_BF16, seed=9, rows=35, k=k, n=40, std=0.1)
    x = wl.make_input(m, 1)
    x[0, 11, :] = np.inf
    os.environ["ECLIP_GEMM_FORCE"] = "1,4,8"
    try:
        got = run_gpu(m, x)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
    rows = np.delete(got.reshape(35, 40), 11, axis=0)
    assert np.isfinite(rows).all() and not np.isfinite(got.reshape(35, 40)[11]).any()
    x[0, 11, :] = 0
    exp = np.delete(orc.run_model(m, x).reshape(35, 40), 11, axis=0)
    assert rel_to_range(rows, exp) <= 2e-4


@pytest.mark.parametrize("cin,cout,groups,k,stride,h,w,batch", [
    (64, 64, 2, 7, 1, 9, 8, 2),           # 49 taps: the general form
    (64, 64, 2, 5, 2, 9, 8, 2),           # 25 taps
    (192, 240, 1 * 3, 1, 1, 7, 9, 3),     # 64 -> 80 channels per group: five tile columns of 16
    (96, 96, 3, 3, 1, 5, 6, 1),           # 32 -> 32 channels per group
    (480, 128, 4, 1, 1, 7, 7, 2),         # one super-group of 480 channels
])
@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
def test_grouped(cin, cout, groups, k, stride, h, w, batch, dt):
    m = wl.single_layer("conv", dt, seed=k + cin, cin=cin, cout=cout, h=h, w=w, k=k, stride=stride, pad=k // 2, groups=groups, act=wl.ACT_RELU,
                        bias_std=0.5)
    x = wl.make_input(m, batch)
    got = run_gpu(m, x)
    assert np.isfinite(got).all()
    assert rel_to_range(got, orc.run_model(m, x)) <= (2.0 ** -8 if dt == wl.DT_BF16 else 2.0 ** -11)
