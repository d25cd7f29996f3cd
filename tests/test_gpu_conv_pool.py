"""A convolution with ReLU and the 2 x 2 max-pool behind it in one launch (copied tiles and the patch kernel), bit for bit against two launches and against the
oracle: every copied tile, patch tiles of each size, even and odd images, a mask that is dealt, and chains that must stay apart."""
from __future__ import annotations

import os

import numpy as np
import pytest

import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


def _model(dt, cin, cout, h, w, k=3, stride=1, pad=1, act=wl.ACT_RELU, pool=(2, 2, 0), seed=1):
    b = graphs._Builder("pooled", dt, seed, graphs.IN_IMAGE, cin, h, w)
    x = b.conv(-1, cin, 1, act=wl.ACT_RELU, bias_std=0.3)
    x = b.conv(x, cout, k, stride, pad, act, bias_std=0.5)
    x = b.maxpool(x, *pool)
    b.conv(x, 16, 1, bias_std=0.3)
    return b.finish()


def _run(g, x, plan, apart):
    if plan: os.environ["ECLIP_GEMM_FORCE"] = plan
    if apart: os.environ["ECLIP_NO_PAIRS"] = "1"
    try:
        return g.run(x, table=[0] * g.m.n_groups), g.h.profile_group_served(0, 0, x.shape[0], 1)[1]
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
        os.environ.pop("ECLIP_NO_PAIRS", None)


def _check(m, batch, plan, fused=True, pool=None):
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch, pool=pool)
    g.m = m
    try:
        one, n_one = _run(g, x, plan, False)
        two, n_two = _run(g, x, plan, True)
    finally:
        g.free()
    assert n_two - n_one == (1 if fused else 0)
    assert np.array_equal(one, two)
    assert rel_to_range(one, orc.run_model(m, x)) <= (2.0 ** -6 if m.dtype == wl.DT_BF16 else 2.0 ** -9)       # three roundings to 16 bits in a row


@pytest.mark.parametrize("tile", range(17, 32))
@pytest.mark.parametrize("dt,cin,cout,h,w,batch", [(wl.DT_BF16, 64, 264, 14, 18, 2), (wl.DT_F16, 64, 72, 9, 11, 3), (wl.DT_BF16, 128, 128, 2, 3, 1)])
def test_copied_tiles(tile, dt, cin, cout, h, w, batch):
    _check(_model(dt, cin, cout, h, w), batch, f"0,{tile},1")


@pytest.mark.parametrize("variant,nw", [(0, 2), (1, 2), (2, 4), (3, 2), (4, 2), (5, 8)])
@pytest.mark.parametrize("h,w", [(12, 16), (9, 7), (3, 2)])
def test_patch_kernel(variant, nw, h, w):
    _check(_model(wl.DT_BF16, 64, 64, h, w), 2, f"2,{variant},{nw}")


def test_strided_and_wider_windows():
    _check(_model(wl.DT_F16, 64, 64, 21, 17, k=5, stride=2, pad=2), 2, "0,26,1")
    _check(_model(wl.DT_BF16, 64, 64, 21, 18, stride=2), 2, "2,0,2")


def test_unequal_shader_engines():
    bits = [32 * cu + 8 * se + xcd for se, n in enumerate((4, 1, 1, 0)) for cu in range(n) for xcd in range(8)]
    pool = ec.Pool([(ec.words_of_bits(bits, 8), 0)])
    try:
        _check(_model(wl.DT_BF16, 64, 128, 62, 64), 2, "0,22,1", pool=pool)
    finally:
        pool.destroy()


@pytest.mark.parametrize("kw", [dict(act=wl.ACT_RELU6), dict(act=wl.ACT_NONE), dict(pool=(2, 1, 0)), dict(pool=(2, 2, 1)), dict(pool=(3, 2, 1))])
def test_other_activations_and_pools_stay_apart(kw):
    _check(_model(wl.DT_BF16, 64, 64, 12, 14, **kw), 2, "0,26,1", fused=False)


def test_a_second_reader_keeps_the_convolution():
    b = graphs._Builder("read twice", wl.DT_BF16, 2, graphs.IN_IMAGE, 64, 12, 12)
    x = b.conv(-1, 64, 1, bias_std=0.3)
    x = b.conv(x, 64, 3, 1, 1, wl.ACT_RELU, bias_std=0.5)
    p = b.maxpool(x, 2, 2, 0)
    b.conv(x, 64, 3, 2, 1, res=p)
    _check(b.finish(), 2, "0,26,1", fused=False)
