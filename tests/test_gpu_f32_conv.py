"""float32 convolutions: every split of a sum among wavefronts and both widths of the loads, and what a layer with many outputs takes."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2506_12598_amd as ec
import workloads as wl
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range, shared_pool

pytestmark = pytest.mark.gpu


def _waves(g, batch, mask_id):
    i, L = g.h.kernel_info(0, mask_id, batch), g.model.layers[0]
    assert i["kernel"] == "conv_f32_kernel"
    return i["workgroups"] * i["threads"] / 64, -(-batch * L.c * L.h * L.w // 64)


@pytest.mark.parametrize("cin,cout,h,w,k,s,p,batch,waves", [
    (16, 96, 40, 37, 1, 1, 0, 1, 1),      # short sums, channels in fours
    (24, 9, 11, 13, 1, 1, 0, 2, 2),
    (12, 20, 9, 8, 2, 1, 1, 1, 4),        # twelve channels: eight and four at a time; padding wider than half the window
    (16, 32, 16, 16, 3, 1, 1, 1, 8),
    (20, 7, 10, 9, 5, 2, 2, 1, 16),
    (64, 64, 30, 30, 3, 1, 1, 8, 4),      # enough outputs on 32 CUs: only as many wavefronts as the length of the sum pays for
    (1, 3, 8, 9, 3, 1, 1, 1, 2),          # one channel at a time
    (3, 16, 9, 7, 3, 2, 1, 2, 4),
    (7, 11, 9, 7, 3, 1, 1, 1, 8),
    (33, 7, 8, 6, 3, 1, 1, 1, 16),
    (6, 40, 60, 60, 5, 1, 2, 2, 4),
])
def test_conv(cin, cout, h, w, k, s, p, batch, waves):
    m = wl.single_layer("conv", wl.DT_F32, seed=cin + cout, cin=cin, cout=cout, h=h, w=w, k=k, stride=s, pad=p, act=wl.ACT_RELU, bias_std=0.5)
    x = wl.make_input(m, batch)
    exp = orc.run_model(m, x)
    g = GpuModel(m, max_batch=batch)
    try:
        mask_id = 1 if batch == 8 else 0
        per_wg = max(1, 4 // waves)                               # sums per workgroup; the last workgroup may be part empty
        n, sums = _waves(g, batch, mask_id)
        assert n == waves * per_wg * -(-sums // per_wg)
        got = g.run(x, table=[mask_id] * m.n_groups)
    finally:
        g.free()
    assert rel_to_range(got, exp) <= 2e-6


def test_many_outputs_take_one_wavefront_each():
    m = wl.single_layer("conv", wl.DT_F32, cin=64, cout=256, h=56, w=56, k=1)
    g = GpuModel(m, max_batch=8)
    try:
        for mask_id in (0, 1):
            n, sums = _waves(g, 8, mask_id)
            assert n == sums
    finally:
        g.free()


def test_padding_never_meets_the_weights():
    # a tap outside the image is no term of the sum, not a term 0 * w
    m = wl.single_layer("conv", wl.DT_F32, seed=5, cin=8, cout=12, h=6, w=7, k=3, pad=1, bias_std=0.5)
    L = m.layers[0]
    x = wl.make_input(m, 1)
    exp = orc.run_model(m, x)
    m.weights[L.w_off:L.w_off + 12 * 8 * 9].reshape(12, 8, 3, 3)[:, :, 0, 0] = np.inf
    g = GpuModel(m)
    try:
        got = g.run(x)
    finally:
        g.free()
    edge = np.zeros(exp.shape, bool)
    edge[:, :, 0, :] = edge[:, :, :, 0] = True                # the outputs that the infinite corner tap is no term of
    assert np.abs(got - exp)[edge].max() <= 2e-6 * (exp.max() - exp.min())
    assert not np.isfinite(got[~edge]).any()


def test_input_that_is_not_16_byte_aligned():
    m = wl.single_layer("linear", wl.DT_F32, seed=6, rows=5, k=64, n=48, bias_std=0.3, std=0.1)
    x = wl.make_input(m, 1)
    buf = torch.zeros(x.size + 4, device="cuda")
    h = ec.Model(shared_pool(), m, m.weights.astype(np.float32), max_batch=1)
    try:
        h.alloc_set([0])
        for shift in range(4):
            buf[shift:shift + x.size] = torch.from_numpy(np.ascontiguousarray(x, dtype=np.float32)).reshape(-1).cuda()
            out = torch.full(m.out_shape(1), float("nan"), device="cuda")
            torch.cuda.synchronize()
            h.submit(buf.data_ptr() + 4 * shift, out.data_ptr(), 1).wait()
            assert rel_to_range(out.cpu().numpy().astype(np.float64), orc.run_model(m, x)) <= 2e-6
    finally:
        h.free()
