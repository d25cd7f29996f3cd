"""Attention whose wavefronts share the keys of 16 queries: ragged key and query blocks, wavefronts without a key, both head sizes, peaked rows."""
from __future__ import annotations

import numpy as np
import pytest

import workloads as wl
from oracle import forward as orc
from gpu_util import GpuModel, rel_to_range

pytestmark = pytest.mark.gpu


def _batch_of_the_other_kernel(seq, heads):
    """Samples from which 32 CUs no longer share the keys: more than 3 workgroups of 16 queries per CU up to 128 keys, more than 2 beyond."""
    return 32 * (3 if seq <= 128 else 2) // (heads * -(-seq // 16)) + 1


def _check_form(g, table, batch, seq, heads, shared):
    i = g.h.kernel_info(0, table, batch)
    queries, threads = (16, 256 if seq <= 128 else 512) if shared else (64, 256)
    assert (i["workgroups"], i["threads"]) == (batch * heads * -(-seq // queries), threads)


@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("seq,hidden,heads,batch", [(1, 64, 1, 1), (15, 64, 2, 2), (33, 192, 3, 1), (65, 128, 4, 2), (97, 256, 4, 1), (128, 128, 2, 4),
                                                    (129, 64, 1, 3), (159, 64, 2, 1), (201, 128, 2, 2), (225, 128, 4, 1), (256, 64, 1, 2)])
@pytest.mark.parametrize("peaked", [False, True])
def test_shared_keys(seq, hidden, heads, batch, peaked, dt):
    m = wl.single_layer("attention", dt, seed=seq + hidden, seq=seq, hidden=hidden, heads=heads)
    x = wl.make_input(m, batch)
    if peaked:                                   # most of a row's weight on keys of one wavefront, another one's for every other query
        x[:, :, :2 * hidden] *= 4.0
        x[:, ::2, :hidden] += 1.5
        x[:, seq // 2:, hidden:2 * hidden] += 1.5
        x = wl.round_to_dtype(x.astype(np.float32), dt)
    exp = orc.run_model(m, x)
    n = _batch_of_the_other_kernel(seq, heads)
    again = np.arange(max(n, batch)) % batch
    g = GpuModel(m, max_batch=len(again))
    try:
        _check_form(g, 5, batch, seq, heads, True)
        _check_form(g, 1, len(again), seq, heads, False)
        few, many = g.run(x, table=[5]), g.run(x[again], table=[1])       # 256 CUs, 32 CUs: two kernels
    finally:
        g.free()
    # probabilities and values are rounded to 16 bits, float32 throughout otherwise: the bound of the other attention tests
    for got, ref in ((few, exp), (many, exp[again])):
        assert np.isfinite(got).all() and rel_to_range(got, ref) <= 6e-3


@pytest.mark.parametrize("dt", [wl.DT_BF16, wl.DT_F16])
@pytest.mark.parametrize("seq", [33, 64, 65, 97, 128, 129, 161, 225, 256])
def test_a_share_of_keys_without_weight(seq, dt):
    """All keys of one wavefront's share score -inf (an infinite element, as a projection that overflowed leaves it): they weigh nothing, whichever share it is."""
    hidden, heads = 128, 2
    m = wl.single_layer("attention", dt, seed=seq, seq=seq, hidden=hidden, heads=heads)
    x0 = np.array(wl.make_input(m, 1))
    x0[:, :, 0:hidden:64] = wl.round_to_dtype(np.abs(x0[:, :, 0:hidden:64]).astype(np.float32) + 0.25, dt)      # the element that meets the infinite one
    n = _batch_of_the_other_kernel(seq, heads)
    g = GpuModel(m, max_batch=n)
    try:
        _check_form(g, 5, 1, seq, heads, True)
        _check_form(g, 1, n, seq, heads, False)
        for first in range(0, seq, 32):
            x = x0.copy()
            x[:, first:first + 32, hidden:2 * hidden:64] = -np.inf
            exp = orc.run_model(m, x)
            assert np.isfinite(exp).all()
            for table, batch in ((5, 1), (1, n)):                # 256 CUs, 32 CUs: two kernels
                got = g.run(np.repeat(x, batch, axis=0), table=[table])
                assert np.isfinite(got).all() and rel_to_range(got, np.repeat(exp, batch, axis=0)) <= 6e-3, (first, table)
    finally:
        g.free()


# 12 heads: the most workgroups per CU that share the keys, and one sample more
@pytest.mark.parametrize("seq,batch,table", [(128, 4, 3), (256, 1, 3), (129, 3, 4), (100, 9, 5)])
def test_where_the_line_lies(seq, batch, table):
    m = wl.single_layer("attention", wl.DT_F16, seed=seq, seq=seq, hidden=768, heads=12)
    x = wl.make_input(m, batch + 1)
    exp = orc.run_model(m, x)
    g = GpuModel(m, max_batch=batch + 1)
    try:
        for b, shared in ((batch, True), (batch + 1, False)):
            _check_form(g, table, b, seq, 12, shared)
            assert rel_to_range(g.run(x[:b], table=[table]), exp[:b]) <= 6e-3
    finally:
        g.free()
