"""Forms of the LDS-tiled GEMM kernels that the layers of the other tests do not reach, every tile forced in turn."""
from __future__ import annotations

import os

import numpy as np
import pytest
import torch

import paper_2506_12598_amd as ec
import workloads as wl
import workloads.graphs as graphs
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range, run_gpu

pytestmark = pytest.mark.gpu

PINGPONG, COPIED = [3, 8, 13, 16], [17, 20, 22, 26, 27]


@pytest.fixture
def force():
    def _force(variant, splits=1):
        os.environ["ECLIP_GEMM_FORCE"] = f"0,{variant},{splits}"
    yield _force
    os.environ.pop("ECLIP_GEMM_FORCE", None)


@pytest.mark.parametrize("variant", PINGPONG + COPIED)
def test_windows_of_more_than_32_taps(variant, force):
    # 49 taps of one K step, 36 of two (four), 36 whose channels the K step of 64 does not divide
    force(variant)
    for i, (cin, kh) in enumerate(((64, 7), (128, 6), (72, 6))):
        m = wl.single_layer("conv", wl.DT_BF16, seed=200 + i, cin=cin, cout=72, h=13, w=11, k=kh, stride=1 + i % 2, pad=3, act=wl.ACT_RELU, bias_std=0.5)
        x = wl.make_input(m, 2)
        assert rel_to_range(run_gpu(m, x), orc.run_model(m, x)) <= 2.0 ** -8


def _dense_block(growth, dtype):
    """Convolutions that read the first channels of a wider tensor (1 x 1 and 3 x 3 windows) and write a channel range of it."""
    b = graphs._Builder("block", dtype, 31, graphs.IN_IMAGE, 16, 17, 15)
    c = b.conv(-1, 64, 3, 1, 1, wl.ACT_RELU, bias_std=0.3)
    for k in (1, 3, 1):
        y = b.conv(c, 128, k, 1, k // 2, wl.ACT_RELU, bias_std=0.3)
        c = b.concat(c, b.conv(y, growth, 3, 1, 1, wl.ACT_RELU6, bias_std=0.3))
    b.gap(c)
    return b.finish()


@pytest.mark.parametrize("growth,dtype", [(64, wl.DT_BF16), (24, wl.DT_F16)])
@pytest.mark.parametrize("variant,splits", [(v, 1) for v in PINGPONG + COPIED + [18, 19, 21, 23, 24, 25, 28]] + [(20, 3), (23, 2)])
def test_row_pitches(variant, splits, growth, dtype, force):
    # concatenation in place: the operand has the pitch of the wider tensor, and so has the output; same bits as with copies
    force(variant, splits)
    m = _dense_block(growth, dtype)
    x = wl.make_input(m, 3)
    got = run_gpu(m, x)
    os.environ["ECLIP_CONCAT_COPY"] = "1"
    try:
        assert np.array_equal(got, run_gpu(m, x))
    finally:
        os.environ.pop("ECLIP_CONCAT_COPY", None)
    assert rel_to_range(got, orc.run_model(m, x)) <= 2e-2


# ---- masks whose shader engines hold different numbers of compute units -------------------------------------------
SHARES = [(8, 8, 2, 2), (5, 8, 3, 1), (1, 0, 0, 8)]


def _bits(share):
    return [32 * cu + 8 * se + xcd for se, n in enumerate(share) for cu in range(n) for xcd in range(8)]


@pytest.fixture(scope="module")
def pools():
    made = {share: ec.Pool([(ec.words_of_bits(_bits(share), 8), 0), (ec.eclip_mask_layout(256, 32, 1, 0, 2), 0)]) for share in SHARES}
    yield made
    for p in made.values():
        p.destroy()


@pytest.mark.parametrize("share", SHARES)
@pytest.mark.parametrize("variant,rows,n", [(17, 700, 2600), (18, 1300, 1300), (20, 1000, 1400), (22, 700, 520), (23, 1100, 700), (24, 600, 3000),
                                            (26, 600, 900), (27, 2300, 1500), (28, 300, 300)])
def test_copied_tiles_are_dealt(variant, rows, n, share, pools, force):
    # grids below, at and above one workgroup per compute unit; other launches leave the rotation in the middle
    force(variant)
    m = wl.single_layer("linear", wl.DT_BF16, seed=rows, rows=rows, k=192, n=n, bias_std=0.3, std=0.05)
    x = wl.make_input(m, 1)
    exp = orc.run_model(m, x)
    g = GpuModel(m, pool=pools[share])
    try:
        for turn in range(4):
            got = g.run(x, table=[0] * m.n_groups)
            assert np.abs(got - exp).max() <= 1e-3 * (exp.max() - exp.min())
            pools[share].probe(1, 5 + turn)
    finally:
        g.free()


@pytest.mark.parametrize("share", SHARES)
def test_captured_requests_on_uneven_masks(share, pools):
    # a captured launch keeps the half of the dealing's notes that it was captured with, whichever half was written last
    m = wl.bert(2, 256, 4, 1024, 201, vocab=500, seed=3, dtype=wl.DT_BF16)
    xs = [wl.make_input(m, 5, seed=40 + i) for i in range(2)]
    between = wl.single_layer("linear", wl.DT_BF16, seed=9, rows=1300, k=192, n=1300, std=0.05)
    xb = wl.make_input(between, 1)
    g, gb = GpuModel(m, max_batch=5, pool=pools[share]), GpuModel(between, pool=pools[share])
    try:
        assert {g.h.kernel_info(i, 0, 5)["kernel"] for i in range(len(m.layers))} & {"conv_gemm_dma_kernel", "conv_gemm_kernel"}
        ref, ref_b = [g.run(x, table=[0] * m.n_groups) for x in xs], gb.run(xb, table=[0] * between.n_groups)
        g.h.graphs(True)
        ids = [torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda() for x in xs]
        outs = [torch.zeros(m.out_shape(5), device="cuda") for _ in xs]
        torch.cuda.synchronize()
        for turn in range(5):
            for i, x in enumerate(ids):
                outs[i].zero_()
                torch.cuda.synchronize()
                g.h.submit(x.data_ptr(), outs[i].data_ptr(), 5).wait()
                assert np.array_equal(outs[i].cpu().numpy().astype(np.float64), ref[i]), (turn, i)
            pools[share].probe(1, 5 + turn)
            assert np.array_equal(gb.run(xb), ref_b)          # one dealt launch on the same stream: the halves change roles
    finally:
        g.free()
        gb.free()


@pytest.mark.parametrize("rows,n,k,kernel", [(1536, 4096, 1024, "conv_gemm_dma_kernel"), (1500, 4088, 1024, "conv_gemm_dma_kernel"),
                                             (1536, 4092, 1024, "conv_gemm_kernel")])
def test_layers_planned_on_256x256_tiles_run_on_the_copied_kernel(rows, n, k, kernel):
    # one tile per CU of 96; ragged rows and columns; columns that the copied kernel's fast epilogue does not take
    pool = ec.Pool([(ec.eclip_mask_layout(256, 32, 1, 0, 3), 0)])
    m = wl.single_layer("linear", wl.DT_BF16, seed=n, rows=rows, k=k, n=n, bias_std=0.3, std=0.05)
    x = wl.make_input(m, 1)
    exp = orc.run_model(m, x)
    g = GpuModel(m, pool=pool)
    try:
        assert g.h.kernel_info(0, 0, 1)["kernel"] == kernel
        assert np.abs(g.run(x, table=[0] * m.n_groups) - exp).max() <= 1e-3 * (exp.max() - exp.min())
    finally:
        g.free()
        pool.destroy()
