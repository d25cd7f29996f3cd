"""Launches on CU masks whose shader engines hold different numbers of compute units: every workgroup's work is done once,
whatever order the shader engines take their turns in (other streams dispatch in between), for tile counts below, at and
above one workgroup per compute unit."""
from __future__ import annotations

import os

import numpy as np
import pytest

import workloads as wl
import paper_2506_12598_amd as ec
from gpu_util import GpuModel
from oracle import forward as orc

pytestmark = pytest.mark.gpu

# enabled CUs of the four shader engines of every XCD
SHARES = [(8, 8, 2, 2), (8, 8, 1, 0), (5, 8, 3, 1), (7, 7, 7, 6), (1, 0, 0, 8)]
_pools = {}


def _pool(share):
    if share not in _pools:
        bits = [32 * cu + 8 * se + xcd for se, n in enumerate(share) for cu in range(n) for xcd in range(8)]
        _pools[share] = ec.Pool([(ec.words_of_bits(bits, 8), 0), (ec.eclip_mask_layout(256, 32, 1, 0, 2), 0)])
    return _pools[share]


@pytest.fixture(scope="module", autouse=True)
def _cleanup():
    yield
    for p in _pools.values():
        p.destroy()


def _check(model, batch, tol, share):
    pool = _pool(share)
    x = wl.make_input(model, batch, dist="normal")
    exp = orc.run_model(model, x)
    g = GpuModel(model, max_batch=batch, pool=pool)
    try:
        for turn in range(4):
            got = g.run(x, table=[0] * model.n_groups)
            assert np.isfinite(got).all()
            assert np.abs(got - exp).max() <= tol * (exp.max() - exp.min())
            pool.probe(1, 5 + turn)                     # workgroup counts that leave the rotation in the middle
    finally:
        g.free()


@pytest.mark.parametrize("share", SHARES)
@pytest.mark.parametrize("force,rows,n", [("0,8,1", 1000, 520), ("0,13,1", 700, 1100), ("0,5,1", 300, 300), ("0,14,2", 1200, 600),
                                          ("0,0,1", 2300, 1500), ("0,9,1", 4100, 1300)])
def test_gemm_tiles(force, rows, n, share):
    os.environ["ECLIP_GEMM_FORCE"] = force
    try:
        m = wl.single_layer("linear", wl.DT_BF16, seed=rows, rows=rows, k=1024 if force.endswith("2") else 192, n=n, bias_std=0.3, std=0.05)
        _check(m, 1, 1e-3, share)
    finally:
        os.environ.pop("ECLIP_GEMM_FORCE", None)


@pytest.mark.parametrize("share", SHARES[:3])
@pytest.mark.parametrize("seq,batch", [(201, 5), (33, 2), (300, 3), (512, 1)])
def test_attention(seq, batch, share):
    m = wl.bert(1, 256, 4, 512, seq, vocab=500, seed=seq, dtype=wl.DT_F16)
    _check(m, batch, 2e-2, share)
