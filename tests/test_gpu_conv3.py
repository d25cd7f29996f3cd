"""The 3 x 3 kernel that works from an image patch in LDS: every tile and number of wavefronts at the sizes where it can go wrong."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu

# images smaller than a tile, whole tiles, remainders of 1 to 3 pixels; channels for idle wavefronts and for several slices each
SHAPES = [(1, 1, 64, 16, 1, 1), (3, 2, 96, 48, 1, 2), (7, 7, 512, 32, 1, 1), (8, 8, 128, 64, 1, 3), (13, 9, 64, 96, 1, 2), (2, 11, 160, 32, 2, 2), (17, 16, 64, 32, 2, 1),
          (9, 14, 256, 64, 2, 1), (5, 6, 544, 32, 1, 1)]


def fits(shape, variant, nw):
    h, w, c, n, stride, batch = shape
    th, tw = ((4, 4), (8, 4), (8, 8))[variant >> 1]
    copies = (((th - 1) * stride + 3) * ((tw - 1) * stride + 3) * 4 + 63) // 64
    slices, bn = c // 32, 32 if variant & 1 else 16
    if slices > nw and (nw < 8 or slices > 4 * nw or (nw == 16 and variant == 5)):
        return False
    return n % bn == 0 and slices > nw // 2 and nw * max(-(-slices // nw) * copies, th * tw * bn // 256) <= 128


def forced(m, x, layer, variant, nw):
    os.environ["ECLIP_GEMM_FORCE"] = f"2,{variant},{nw}"
    try:
        g = GpuModel(m, max_batch=x.shape[0])
        try:
            assert g.h.kernel_info(layer, 0, x.shape[0])["kernel"] == "conv3_kernel"
            return g.run(x)
        finally:
            g.free()
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)


@pytest.mark.parametrize("shape,variant,nw", [(s, v, nw) for s in SHAPES for v in range(6) for nw in (2, 4, 8, 16) if fits(s, v, nw)])
def test_tiles(shape, variant, nw):
    h, w, c, n, stride, batch = shape
    m = wl.single_layer("conv", wl.DT_F16 if c % 64 else wl.DT_BF16, seed=h * w + c, cin=c, h=h, w=w, cout=n, k=3, stride=stride, pad=1, act=wl.ACT_RELU, bias_std=0.3)
    x = wl.make_input(m, batch)
    got = forced(m, x, 0, variant, nw)
    # float32 sums of 9 c products, stored in 16 bits: 2^-9 of a value, and a value is at most the range
    assert np.isfinite(got).all() and rel_to_range(got, orc.run_model(m, x)) <= 2.0 ** -8


@pytest.mark.parametrize("variant,nw", [(0, 2), (3, 2), (4, 2)])
@pytest.mark.parametrize("act", [wl.ACT_NONE, wl.ACT_RELU6, wl.ACT_GELU])
def test_residual_and_channel_ranges(variant, nw, act):
    # reads the first 64 channels of a wider buffer with that buffer's pitch, adds a residual, and writes a channel range of another
    b = graphs._Builder("ranges", wl.DT_F16, 7 + act, graphs.IN_IMAGE, 8, 11, 6)
    x = b.conv(-1, 64, 1, bias_std=0.3)
    t = b.conv(x, 64, 3, 1, 1, act, res=x, bias_std=0.3)
    y = b.concat(t, b.conv(t, 32, 3, 1, 1, act, bias_std=0.3))
    z = b.conv(y, 32, 3, 1, 1, bias_std=0.3)
    b.linear(b.gap(b.concat(y, z)), 24, std=0.1)
    m = b.finish()
    x_in = wl.make_input(m, 2)
    got = forced(m, x_in, t, variant, nw)
    # four layers stored in float16, 2^-12 of a value each and magnified by no more than 2 in the next: the bound is 16 of them
    assert np.isfinite(got).all() and rel_to_range(got, orc.run_model(m, x_in)) <= 2.0 ** -8


# grouped: super-groups of 32 input channels with 16, 32 and 64 outputs; more tiles than a workgroup's four, and fewer
@pytest.mark.parametrize("h,w,cin,cout,groups,stride,batch", [(1, 1, 64, 64, 16, 1, 1), (7, 9, 128, 128, 32, 1, 3), (13, 4, 64, 128, 8, 1, 2), (9, 17, 64, 32, 8, 2, 1),
                                                              (16, 8, 96, 96, 3, 2, 2), (5, 5, 32, 32, 8, 1, 1)])
@pytest.mark.parametrize("blocks", [1, 2, 4])
@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
def test_grouped(h, w, cin, cout, groups, stride, batch, blocks, dt):
    m = wl.single_layer("conv", dt, seed=h + cin + cout, cin=cin, cout=cout, h=h, w=w, k=3, stride=stride, pad=1, groups=groups, act=wl.ACT_RELU, bias_std=0.4,
                        residual=True)
    x = wl.make_input(m, batch)
    os.environ["ECLIP_GCONV3"] = str(blocks)
    try:
        g = GpuModel(m, max_batch=batch)
        try:
            info = g.h.kernel_info(1, 0, batch)
            th, tw = (4, 8, 8)[blocks // 2], (4, 4, 8)[blocks // 2]
            ho, wo = (h - 1) // stride + 1, (w - 1) // stride + 1
            columns = cout // (32 if cout * 32 // cin % 32 == 0 else 16)
            assert info["kernel"] == "gconv_mfma_kernel" and info["workgroups"] == -(-batch * -(-ho // th) * -(-wo // tw) * columns // 4)
            got = g.run(x)
        finally:
            g.free()
    finally:
        del os.environ["ECLIP_GCONV3"]
    # two layers stored in 16 bits, 2^-9 (2^-12) of a value each
    assert np.isfinite(got).all() and rel_to_range(got, orc.run_model(m, x)) <= (2.0 ** -8 if dt == wl.DT_BF16 else 2.0 ** -11)
