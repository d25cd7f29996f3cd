"""The copied tiles of which two workgroups fit a compute unit (128 x 256, 128 x 192, 192 x 128), forced: linear layers and windows, ragged rows and columns,
one K step to many, K in slices, storage and float outputs, residuals, GELU; grids below and beyond two workgroups per unit, on a mask that is dealt too."""
from __future__ import annotations

import os

import numpy as np
import pytest

import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range, run_gpu

pytestmark = pytest.mark.gpu

TILES = {29: (128, 256), 30: (128, 192), 31: (192, 128)}


@pytest.fixture
def force():
    def _force(variant, splits=1):
        os.environ["ECLIP_GEMM_FORCE"] = f"0,{variant},{splits}"
    yield _force
    os.environ.pop("ECLIP_GEMM_FORCE", None)


def _two_layers(dt, rows, k, n, act, storage):
    b = graphs._Builder("layers", dt, 31 * n + k + act, graphs.IN_SEQ, k, 1, rows)
    first = b.linear(-1, n, std=1.0 / np.sqrt(k), bias_std=0.3)
    out = b.linear(-1, n, act=act, res=first, std=1.0 / np.sqrt(k), bias_std=0.5)
    if storage:
        b.eltwise(out)                       # passes the rounded values on as floats
    return b.finish()


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("dt,act,rows,k,n,storage,splits", [
    (wl.DT_BF16, wl.ACT_GELU, 300, 32, 520, True, 1), (wl.DT_F16, wl.ACT_RELU6, 128, 352, 512, True, 1), (wl.DT_F16, wl.ACT_GELU, 193, 64, 264, True, 1),
    (wl.DT_BF16, wl.ACT_GELU, 385, 96, 520, False, 1), (wl.DT_F16, wl.ACT_RELU, 17, 1056, 776, False, 1), (wl.DT_BF16, wl.ACT_NONE, 130, 1536, 200, True, 3),
])
def test_linear_layers(tile, dt, act, rows, k, n, storage, splits, force):
    # Float outputs differ from the oracle by the order of at most 1536 additions (2e-4 of the range as for every linear layer here) and by the
    # residual's one rounding, at most 2^-9 (2^-12) of the larger of the two summands; storage outputs are rounded once more.  Twice that is the bound.
    step = 2.0 ** -9 if dt == wl.DT_BF16 else 2.0 ** -12
    m = _two_layers(dt, rows, k, n, act, storage)
    x = wl.make_input(m, 1)
    force(tile, splits)
    got = run_gpu(m, x)
    assert np.isfinite(got).all()
    assert rel_to_range(got, orc.run_model(m, x)) <= 2 * step * (storage + 1) + 2e-4


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("cin,cout,h,w,k,stride,pad", [(32, 72, 19, 17, 3, 1, 1), (96, 264, 15, 18, 3, 2, 1), (64, 136, 13, 11, 5, 1, 2), (128, 200, 14, 9, 1, 2, 0)])
def test_windows(tile, cin, cout, h, w, k, stride, pad, force):
    m = wl.single_layer("conv", wl.DT_BF16, seed=cin + cout, cin=cin, cout=cout, h=h, w=w, k=k, stride=stride, pad=pad, act=wl.ACT_RELU, bias_std=0.5)
    x = wl.make_input(m, 2)
    force(tile)
    assert rel_to_range(run_gpu(m, x), orc.run_model(m, x)) <= 2.0 ** -8


@pytest.mark.parametrize("tile", TILES)
@pytest.mark.parametrize("cus", [32, 48])                # even, and 8 + 8 + ... dealt to unequal shader engines
def test_grids_beyond_two_per_unit(tile, cus, force):
    bits = [32 * cu + 8 * se + xcd for se, n in enumerate((1, 1, 1, 1) if cus == 32 else (4, 1, 1, 0)) for cu in range(n) for xcd in range(8)]
    pool = ec.Pool([(ec.words_of_bits(bits, 8), 0)])
    m = wl.single_layer("linear", wl.DT_BF16, seed=tile, rows=1000, k=192, n=2600, bias_std=0.3, std=0.05)
    x = wl.make_input(m, 1)
    exp = orc.run_model(m, x)
    force(tile)
    g = GpuModel(m, pool=pool)
    try:
        assert g.h.kernel_info(0, 0, 1)["tile"] == TILES[tile]
        first = g.run(x, table=[0])
        assert np.abs(first - exp).max() <= 1e-3 * (exp.max() - exp.min())
        for _ in range(20):                  # the same bits however the workgroups of a unit fall together
            assert np.array_equal(g.run(x, table=[0]), first)
    finally:
        g.free()
        pool.destroy()


def test_layers_without_a_fast_form_are_left_to_the_planner(force):
    force(29)
    m = wl.single_layer("linear", wl.DT_BF16, seed=3, rows=200, k=72, n=512, bias_std=0.3, std=0.05)
    x = wl.make_input(m, 1)
    g = GpuModel(m)
    try:
        assert g.h.kernel_info(0, 0, 1)["tile"] != (128, 256)
        assert rel_to_range(g.run(x), orc.run_model(m, x)) <= 2e-4
    finally:
        g.free()
