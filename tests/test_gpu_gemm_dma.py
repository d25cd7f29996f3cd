"""Every tile shape of the GEMM kernel that copies its operands straight into LDS, forced in turn: ragged M, N and K, fewer K
steps than ring stages, K slices, and its three ways of addressing the activations."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
from oracle import forward as orc
from gpu_util import rel_to_range, run_gpu

pytestmark = pytest.mark.gpu

CASES = [
    # (layer, batch, tolerance)
    (dict(op="linear", dtype=wl.DT_BF16, rows=300, k=64, n=200, bias_std=0.3, std=0.1), 1, 2e-4),           # one K step
    (dict(op="linear", dtype=wl.DT_F16, rows=517, k=128, n=136, act=wl.ACT_GELU, bias_std=0.3, std=0.1), 1, 3e-4),
    (dict(op="linear", dtype=wl.DT_BF16, rows=1100, k=1024, n=1100, std=0.05), 1, 2e-4),
    (dict(op="linear", dtype=wl.DT_F16, rows=70, k=192, n=76, bias_std=0.3, std=0.1), 3, 3e-4),              # N not a multiple of 8
    (dict(op="linear", dtype=wl.DT_BF16, rows=130, k=72, n=264, bias_std=0.3, std=0.1), 2, 2e-4),            # K not a multiple of 64
    (dict(op="conv", dtype=wl.DT_F16, cin=128, cout=72, h=19, w=17, k=1, stride=2, pad=0, act=wl.ACT_RELU, bias_std=0.5), 2, 2.0 ** -8),
    (dict(op="conv", dtype=wl.DT_BF16, cin=64, cout=40, h=15, w=18, k=3, stride=2, pad=1, bias_std=0.5, residual=True), 2, 2.0 ** -7),
    (dict(op="conv", dtype=wl.DT_BF16, cin=192, cout=200, h=11, w=13, k=3, stride=1, pad=1, act=wl.ACT_RELU, bias_std=0.5), 2, 2.0 ** -8),
    (dict(op="conv", dtype=wl.DT_BF16, cin=24, cout=96, h=20, w=20, k=3, stride=1, pad=1, act=wl.ACT_RELU, bias_std=0.5), 2, 2.0 ** -8),
]


@pytest.mark.parametrize("splits", [1, 3])
@pytest.mark.parametrize("variant", range(17, 29))
def test_tile(variant, splits):
    os.environ["ECLIP_GEMM_FORCE"] = f"0,{variant},{splits}"
    try:
        for i, (kw, batch, tol) in enumerate(CASES):
            kw = dict(kw)
            m = wl.single_layer(kw.pop("op"), kw.pop("dtype"), seed=100 + i, **kw)
            x = wl.make_input(m, batch, dist="normal")
            exp = orc.run_model(m, x)
            got = run_gpu(m, x)
            assert np.isfinite(got).all(), (i, kw)
            assert rel_to_range(got, exp) <= tol, (i, kw)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)
