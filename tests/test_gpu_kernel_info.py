"""eclip_model_kernel_info reports the kernel, the workgroups and the threads that a layer is launched with."""
from __future__ import annotations

import os

import pytest

import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs
from gpu_util import shared_pool

pytestmark = pytest.mark.gpu


def _info(m, batch, mask_id=0):
    h = ec.Model(shared_pool(), m, wl.to_storage(m.weights, m.dtype), max_batch=batch)
    try:
        return h.kernel_info(0, mask_id, batch)
    finally:
        h.free()


@pytest.mark.parametrize("variant,kernel,threads,tile", [
    (0, "conv_gemm_kernel", 256, (128, 128)), (1, "conv_gemm_kernel", 256, (64, 64)),                 # both operands staged by 4 wavefronts
    (3, "conv_gemm_kernel", 512, (256, 256)), (8, "conv_gemm_kernel", 512, (192, 128)), (16, "conv_gemm_kernel", 512, (96, 192)),
    (17, "conv_gemm_dma_kernel", 256, (256, 256)), (20, "conv_gemm_dma_kernel", 256, (128, 128)), (28, "conv_gemm_dma_kernel", 256, (128, 128)),
])
def test_lds_tiles(variant, kernel, threads, tile):
    os.environ["ECLIP_GEMM_FORCE"] = f"0,{variant},1"
    try:
        i = _info(wl.single_layer("linear", wl.DT_BF16, rows=700, k=128, n=900), 1)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
    assert (i["kernel"], i["threads"], i["tile"]) == (kernel, threads, tile)
    assert i["workgroups"] >= -(-700 // tile[0]) * -(-900 // tile[1])


def test_depthwise_workgroups():
    # 100 channels: one element per thread; 64 channels of 200 x 201: strips of 2 x 18 pixels x 8 channels on 32 CUs
    assert _info(wl.single_layer("conv", wl.DT_F16, cin=100, cout=100, h=9, w=7, k=3, pad=1, groups=100), 2)["workgroups"] == -(-2 * 63 * 100 // 256)
    i = _info(wl.single_layer("conv", wl.DT_BF16, cin=64, cout=64, h=200, w=201, k=3, pad=1, groups=64), 2, 1)
    rows = {24: 9, 18: 12, 12: 17, 9: 23}
    assert i["kernel"] == "dwconv3_strip_kernel"
    assert i["workgroups"] in {(-(-2 * r * 101 * 8 // 256) + 7) // 8 * 8 for r in rows.values()}


def _layers_behind_an_image():
    b = graphs._Builder("first", wl.DT_BF16, 3, graphs.IN_IMAGE, 3, 64, 64)
    x = b.conv(-1, 64, 7, 2, 3, act=wl.ACT_RELU)
    b.eltwise(b.maxpool(x, 3, 2, 1))
    return b.finish()


def _depthwise_and_pointwise():
    b = graphs._Builder("dwpw", wl.DT_BF16, 4, graphs.IN_IMAGE, 8, 20, 20)
    x = b.conv(-1, 64, 1)
    b.eltwise(b.conv(b.conv(x, 64, 3, 1, 1, groups=64), 32, 1))
    return b.finish()


@pytest.mark.parametrize("plain", [False, True])
def test_a_first_layer_on_the_callers_planes_is_reported_timed_and_left_out_of_tuning(plain):
    m = _layers_behind_an_image()
    if plain:
        os.environ["ECLIP_NO_PAIRS"] = "1"
    h = ec.Model(shared_pool(), m, wl.to_storage(m.weights, m.dtype), max_batch=2)
    try:
        i = h.kernel_info(0, 5, 2)
        if plain:
            assert i["kernel"] != "stem_kernel"
        else:
            # 32 x 32 outputs in tiles of 4 x 16, since 16 of 8 x 16 would leave CUs without one
            assert (i["kernel"], i["workgroups"], i["threads"], i["tile"], i["mnk"]) == ("stem_kernel", 32, 256, (64, 64), (2048, 64, 147 // 3 * 8))
        assert len(h.profile_group(0, 5, 2, iters=3)) == 3
        assert h.tune(5, batch=2, iters=1) == (1 if plain else 0)
    finally:
        h.free()
        os.environ.pop("ECLIP_NO_PAIRS", None)


@pytest.mark.parametrize("plan,tuned", [("2,2", 1), ("0,0", 2)])
def test_a_pointwise_layer_in_one_launch_with_the_depthwise_is_left_out_of_tuning(plan, tuned):
    m = _depthwise_and_pointwise()
    os.environ["ECLIP_DWPW"] = plan
    h = ec.Model(shared_pool(), m, wl.to_storage(m.weights, m.dtype), max_batch=1)
    try:
        assert h.tune(0, batch=1, iters=1) == tuned and h.tune(0, batch=1, iters=1) == 0
    finally:
        h.free()
        os.environ.pop("ECLIP_DWPW", None)
