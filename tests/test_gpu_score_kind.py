"""The contraction over a tile's vocabulary and the lists it reads, forced where
the plan would sum each target sentence's words: its variants give the same
bits, and S meets the oracle's bars."""
import numpy as np
import pytest

import oracle
from synth import corpus
from tests import helpers as H
from tests.test_gpu_parity import _fused_edge_batch, _varying_degree_batch, _wide_vocabulary_batch

pytestmark = pytest.mark.gpu

BATCHES = {"ragged": lambda: corpus.make_batch(2, pairs=40), "fused edges": _fused_edge_batch,
           "wide vocabulary": _wide_vocabulary_batch, "varying degree": _varying_degree_batch}
DENSE = {"score_kind": 1}


def _dense(b, prec, **params):
    r = H.run_gpu(b, prec=prec, params=dict(DENSE, **params), timing=True)
    assert r["miner"].plan.score_cells() == (b.cells(), 0)
    return r


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("batch", sorted(BATCHES))
def test_dense_variants_give_the_same_bits(batch, prec):
    b = BATCHES[batch]()
    one = _dense(b, prec)
    ora = oracle.score(b)
    if prec == 0:
        assert H.s_rel_err(one["S"], ora["S64"]).max() <= 1e-5
    else:
        assert np.abs(one["S"].astype(np.float64) - ora["S64"]).max() <= 2e-2
    H.assert_align_equal(one, oracle.align(b.n, b.m, one["S"], b.gap, b.threshold), b.n, b.m)
    two_kernels = _dense(b, prec, expand_fused=0)
    assert two_kernels["launches"]["build_a"] > 0 and two_kernels["launches"]["expand_a"] == 0
    for other in (two_kernels, _dense(b, prec, score_kgroup=2), _dense(b, prec, score_xcd_map=0)):
        for k in ("S", "S_raw"):
            np.testing.assert_array_equal(other[k].view(np.uint32), one[k].view(np.uint32))


@pytest.mark.parametrize("batch", ["ragged", "fused edges"])
def test_fp32_kinds_add_in_one_order(batch):
    # each target sentence's own words, a tile's, the whole vocabulary: the same
    # FP32 additions, the others add zeros between them
    b = BATCHES[batch]()
    summed = H.run_gpu(b, prec=0)
    assert summed["miner"].plan.score_cells() == (0, b.cells())
    for other in (_dense(b, 0), H.run_gpu(b, prec=0, params={"score_compact": 0})):
        for k in ("S", "S_raw"):
            np.testing.assert_array_equal(other[k].view(np.uint32), summed[k].view(np.uint32))


def test_kinds_are_counted():
    import paper_1512_01641_amd as nw
    b = corpus.make_batch(2, pairs=40)
    mn = nw.Miner(nw.Context(0), nw.DeviceBatch.from_host(b), nw.DeviceDict.from_host(b), nw.NWM_FP32)
    assert mn.plan.score_cells() == (0, b.cells())
    for name, value, want in (("score_kind", 1, (b.cells(), 0)), ("score_kind", 2, (0, b.cells())),
                              ("score_compact", 0, (b.cells(), 0))):
        mn.plan.set_param(name, value)
        assert mn.plan.score_cells() == want
    with pytest.raises(nw.NwmError):
        mn.plan.set_param("score_kind", 3)
