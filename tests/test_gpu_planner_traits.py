"""Layers that fill a share whose shader engines hold unequal numbers of compute units run on tiles that are dealt to the engines."""
from __future__ import annotations

import numpy as np
import pytest

import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cus", [144, 160, 192])                # 8 + 8 + 1 + 1, 8 + 8 + 2 + 2 and 8 + 8 + 4 + 4 CUs per XCD
@pytest.mark.parametrize("kw,batch,tol", [
    (dict(op="linear", dtype=wl.DT_BF16, rows=1005, k=3072, n=768, bias_std=0.3, std=0.02), 1, 2e-4),      # float32 output
    (dict(op="conv", dtype=wl.DT_F16, cin=128, cout=128, h=28, w=28, k=3, stride=1, pad=1, act=wl.ACT_RELU, bias_std=0.5), 3, 2.0 ** -11),
])
def test_dealt_tiles(cus, kw, batch, tol):
    kw = dict(kw)
    pool = ec.Pool([(ec.eclip_mask_layout(256, 16, 1, 0, cus // 16), 0)])
    m = wl.single_layer(kw.pop("op"), kw.pop("dtype"), seed=cus, **kw)
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch, pool=pool)
    try:
        assert g.h.kernel_info(0, 0, batch)["kernel"] in ("conv_gemm_dma_kernel", "conv_gemm_kernel")
        got = g.run(x, table=[0] * m.n_groups)
        assert np.isfinite(got).all()
        assert rel_to_range(got, orc.run_model(m, x)) <= tol
    finally:
        g.free()
        pool.destroy()


def test_tuning_starts_from_the_plan_an_untuned_model_runs():
    # 256 x 256 tiles on 96 CUs: the copied kernel untuned, and no slower kernel of the same tile after tuning (50 us on the ping-pong kernel, 47)
    pool = ec.Pool([(ec.eclip_mask_layout(256, 32, 1, 0, 3), 0)])
    m = wl.single_layer("linear", wl.DT_BF16, seed=5, rows=1536, k=2048, n=4096, std=0.02)
    h = ec.Model(pool, m, wl.to_storage(m.weights, m.dtype))
    try:
        before = h.kernel_info(0, 0, 1)
        assert before["kernel"] == "conv_gemm_dma_kernel" and before["tile"] == (256, 256)
        assert h.tune(0, batch=1, iters=3) == 1
        after = h.kernel_info(0, 0, 1)
        assert after["kernel"] == "conv_gemm_dma_kernel" or after["tile"] != (256, 256)
    finally:
        h.free()
        pool.destroy()


def test_equal_sizes_in_different_address_forms_are_tuned_apart():
    # M = 36, N = 64, K = 288: a 3 x 3 window over 32 channels and a 2 x 2 window over 72, which only the general kernels take
    b = graphs._Builder("twins", wl.DT_BF16, 3, graphs.IN_IMAGE, 64, 6, 6)
    wide = b.conv(-1, 72, 2, 1, 1)
    slim = b.conv(-1, 32, 1)
    p = b.conv(slim, 64, 3, 1, 1)
    q = b.conv(wide, 64, 2)
    b.eltwise(p, res=q)
    m = b.finish()
    x = wl.make_input(m, 1)
    g = GpuModel(m)
    try:
        assert g.h.kernel_info(p, 0, 1)["mnk"] == g.h.kernel_info(q, 0, 1)["mnk"] == (36, 64, 288)
        assert g.h.tune(0, batch=1, iters=1) == 4
        assert g.h.tune(0, batch=1, iters=1) == 0
        assert rel_to_range(g.run(x), orc.run_model(m, x)) <= 2.0 ** -6       # three roundings to bf16 in a row
    finally:
        g.free()
