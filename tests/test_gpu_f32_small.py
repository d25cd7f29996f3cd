"""float32 convolutions that share their sum among wavefronts, and the pool + classifier kernels at the ends of their ranges."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cin,cout,h,w,k,s,p,batch", [
    (1, 1, 3, 3, 1, 1, 0, 1),        # one output position per lane group, K shorter than a wavefront's slice
    (3, 16, 9, 7, 3, 2, 1, 2),       # K = 27 on four wavefronts
    (8, 5, 6, 5, 2, 1, 0, 3),        # K = 32: the last size of that form
    (11, 24, 8, 9, 3, 1, 1, 1),      # K = 99 on eight wavefronts, ragged slices
    (33, 7, 5, 4, 1, 1, 0, 2),       # K = 33: the first size of it; the last wavefront has no work
    (64, 10, 7, 7, 5, 3, 2, 1),
])
def test_conv_f32_reads_either_layout(cin, cout, h, w, k, s, p, batch):
    m = wl.single_layer("stem", wl.DT_F32, seed=cin + cout, cin=cin, cout=cout, h=h, w=w, k=k, stride=s, pad=p, bias_std=0.5)
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch)
    try:
        got, (_, n_k, _) = g.run(x, table=[0], timing=True)
    finally:
        g.free()
    assert n_k == 3                  # the first convolution reads the caller's planes, no re-layout before it
    assert rel_to_range(got, orc.run_model(m, x)) <= 2e-6
    m = wl.single_layer("conv", wl.DT_F32, seed=cin + cout, cin=cin, cout=cout, h=h, w=w, k=k, stride=s, pad=p, act=wl.ACT_RELU,
                        bias_std=0.5, residual=True)
    assert rel_to_range(run_gpu(m, x), orc.run_model(m, x)) <= 2e-6


@pytest.mark.parametrize("dt,c,h,w,n,batch", [
    (wl.DT_F32, 4, 3, 5, 10, 1), (wl.DT_F32, 32, 16, 16, 10, 4), (wl.DT_F32, 1024, 8, 8, 300, 2), (wl.DT_F32, 100, 7, 1, 33, 20),
    (wl.DT_BF16, 8, 3, 3, 17, 2), (wl.DT_F16, 2048, 8, 8, 1000, 1), (wl.DT_BF16, 2048, 1, 7, 40, 8), (wl.DT_F16, 136, 30, 30, 8, 1),
])
def test_pool_and_classifier(dt, c, h, w, n, batch):
    m = wl.single_layer("gapfc", dt, seed=c + n, c=c, h=h, w=w, n=n, act=wl.ACT_RELU, bias_std=0.3, std=1.0 / np.sqrt(c))
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch)
    try:
        got, (_, n_k, _) = g.run(x, table=[0], timing=True)
    finally:
        g.free()
    assert n_k == 2                  # input re-layout, pool + classifier
    assert rel_to_range(got, orc.run_model(m, x)) <= {wl.DT_F32: 2e-6, wl.DT_BF16: 4e-3, wl.DT_F16: 1e-3}[dt]


@pytest.mark.parametrize("dt,c,h,w,n,batch,mask_id,fused", [
    (wl.DT_F32, 512, 7, 7, 1000, 1, 0, True), (wl.DT_F32, 512, 7, 7, 1000, 8, 0, True),      # 32 workgroups per item on 256 CUs
    (wl.DT_F32, 512, 7, 7, 1000, 9, 0, False), (wl.DT_F32, 512, 7, 7, 1000, 2, 1, False),    # ... and on 32
    (wl.DT_F32, 128, 7, 7, 1000, 4, 1, True), (wl.DT_F32, 128, 7, 7, 1000, 5, 1, False),     # small workgroups: four per CU
    (wl.DT_BF16, 2048, 7, 7, 1000, 8, 0, True), (wl.DT_F16, 2048, 7, 7, 1000, 5, 1, True),   # 16 bit: several blocks of 16 outputs per
    (wl.DT_BF16, 512, 7, 7, 1001, 1, 1, True), (wl.DT_F16, 136, 9, 9, 530, 8, 1, True),      # workgroup, their number ragged
    (wl.DT_BF16, 64, 3, 3, 8000, 3, 1, True), (wl.DT_F16, 512, 7, 7, 1000, 9, 0, False),
])
def test_pool_and_classifier_on_few_compute_units(dt, c, h, w, n, batch, mask_id, fused):
    m = wl.single_layer("gapfc", dt, seed=c + n, c=c, h=h, w=w, n=n, bias_std=0.3, std=1.0 / np.sqrt(c))
    x = wl.make_input(m, batch)
    g = GpuModel(m, max_batch=batch)
    try:
        got, (_, n_k, _) = g.run(x, table=[mask_id], timing=True)
    finally:
        g.free()
    assert (n_k == 2) == fused       # input re-layout, pool + classifier
    assert rel_to_range(got, orc.run_model(m, x)) <= {wl.DT_F32: 2e-6, wl.DT_BF16: 4e-3, wl.DT_F16: 1e-3}[dt]
