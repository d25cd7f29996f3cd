"""The caller's output is aligned as floats are and no more: every kernel that writes it as a last layer, at an address four bytes past a multiple of 256."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import workloads as wl
from oracle import forward as orc
from gpu_util import GpuModel, dev_input, rel_to_range

pytestmark = pytest.mark.gpu


LAST = [
    ("layernorm", dict(rows=9, width=256, residual=True, affine_std=0.5), 2), ("softmax", dict(rows=9, width=64), 2),
    ("linear", dict(rows=40, k=64, n=72, bias_std=0.3), 1), ("linear", dict(rows=600, k=512, n=2048, std=0.03, bias_std=0.3), 1),
    ("linear", dict(rows=1536, k=256, n=4096, std=0.05), 1), ("conv", dict(cin=32, cout=40, h=7, w=6, k=3, pad=1, bias_std=0.3), 2),
    ("gap", dict(c=64, h=7, w=7), 3), ("gapfc", dict(c=64, h=7, w=7, n=40, bias_std=0.3), 2), ("eltwise", dict(rows=9, width=64), 2),
    ("attention", dict(hidden=128, heads=2, seq=40), 2),                   # 16-bit types only
]


@pytest.mark.parametrize("op,kw,batch,dt", [c + (wl.DT_BF16,) for c in LAST] + [c + (wl.DT_F32,) for c in LAST if c[0] != "attention"])
def test_float_aligned_output(op, kw, batch, dt):
    m = wl.single_layer(op, dt, seed=11, **kw)
    x = wl.make_input(m, batch)
    exp = orc.run_model(m, x)
    g = GpuModel(m, max_batch=batch)
    try:
        d_in = dev_input(m, x)
        n = int(np.prod(m.out_shape(batch)))
        room = torch.full((n + 128,), 7.0, device="cuda")
        at = -(room.data_ptr() // 4) % 64 + 1
        assert (room.data_ptr() + 4 * at) % 256 == 4
        g.h.submit(d_in.data_ptr(), room.data_ptr() + 4 * at, batch).wait()
        out = room.cpu().numpy()
    finally:
        g.free()
    assert np.all(out[:at] == 7.0) and np.all(out[at + n:] == 7.0)             # nothing around it is touched
    got = out[at:at + n].reshape(exp.shape).astype(np.float64)
    assert rel_to_range(got, exp) <= (1e-5 if dt == wl.DT_F32 else 2.0 ** -7)  # float32 sums; two roundings to bf16
