"""Forms of the LDS-tiled GEMM kernels that the layers of the other tests do not reach, every tile forced in turn."""
from __future__ import annotations

import os

import pytest

import workloads as wl
from oracle import forward as orc
from gpu_util import rel_to_range, run_gpu

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
