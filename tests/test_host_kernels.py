"""The scoring kernels' own sources on the host wave machine, under the address
and undefined-behaviour sanitizers, against the FP64 oracle: the batches of
test_gpu_sparse.py (list lengths around the sorting network and past it, repeated
words, a vocabulary larger than the table, runs of column tiles), parts of one
batch by different contractions, and plans drawn at random."""
import numpy as np
import pytest

import oracle
from tests import helpers as H
from tests import host_machine as M
from tests.test_gpu_sparse import CASES, _batch


@pytest.fixture(scope="session")
def program(tmp_path_factory):
    return M.build(tmp_path_factory.mktemp("host"))


def _bits(x):
    return x.view(np.uint32)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("case", sorted(CASES))
def test_contractions_in_bounds(program, case, prec):
    b = CASES[case]()
    two = M.run(program, b, prec=prec, params={"expand_fused": 0}, apart=True)
    if prec == 0 or case != "table":
        assert two["launches"]["merge"] > 0 and two["launches"]["build_a"] == 0   # the sparse route ran
    one = M.run(program, b, prec=prec, passes=2)
    np.testing.assert_array_equal(_bits(one["S"]), _bits(two["S"]))
    np.testing.assert_array_equal(_bits(one["S_raw"]), _bits(two["S_raw"]))
    quiet = M.run(program, b, prec=prec, raw=False)
    np.testing.assert_array_equal(_bits(quiet["S"]), _bits(one["S"]))
    for order in (1, 2):   # waves and lanes in other orders: no race
        other = M.run(program, b, prec=prec, order=order)
        np.testing.assert_array_equal(_bits(other["S"]), _bits(one["S"]))
    ora = oracle.score(b)
    if prec == 0:
        assert H.s_rel_err(one["S"], ora["S64"]).max() <= 1e-5
    else:
        assert np.abs(one["S"].astype(np.float64) - ora["S64"]).max() <= 2e-2
    if case != "runs":   # (a minute on this machine)
        dense = M.run(program, b, prec=prec, params={"score_compact": 0})
        if prec == 0:   # the same sums in the same order
            np.testing.assert_array_equal(_bits(one["S_raw"]), _bits(dense["S_raw"]))


def test_parts_by_different_contractions_in_bounds(program):
    # a long pair (summed) among short ones (BF16 operands: dense tiles)
    b = _batch([200] + [20, 40, 64] * 4, [700] + [25, 64, 33] * 4, 2048, [5, 22, 40], [5, 22, 40])
    ora = oracle.score(b)
    one = M.run(program, b, prec=1, params={"expand_fused": 0}, apart=True, split=64)
    assert one["launches"]["build_a"] > 0 and one["launches"]["build_a"] < one["launches"]["merge"]
    assert np.abs(one["S"].astype(np.float64) - ora["S64"]).max() <= 2e-2
    mined = M.run(program, b, op="mine", prec=1, passes=2, split=64)
    np.testing.assert_array_equal(_bits(mined["S"]), _bits(one["S"]))


def test_tiles_with_and_without_records(program):
    # a tall narrow pair (dense by the plan's rule, so its tiles have records)
    # before wide ones (summed), then all of them dense by parameter
    b = _batch([1300, 20, 30], [60, 330, 290], 2048, [5, 12], [5, 22, 9], seed=9)
    S = oracle.score(b)["S64"]
    for params in ({}, {"score_kind": 1}, {"score_kind": 2}):
        got = M.run(program, b, prec=1, params=params, split=64)["S"]
        assert np.abs(got.astype(np.float64) - S).max() <= 2e-2


@pytest.mark.parametrize("seed", range(6))
def test_drawn_plans_in_bounds(program, seed):
    rng = np.random.default_rng([41, seed])
    pairs = int(rng.integers(1, 7))
    n = rng.integers(0, 90, pairs)
    m = rng.integers(0, 150, pairs)
    n[0], m[0] = rng.integers(1, 300), rng.integers(1, 300)
    b = _batch(n, m, int(rng.integers(4, 20000)), rng.integers(0, 49, 7), rng.integers(0, [50, 130][seed % 2], 9), seed=seed)
    prec = seed // 2 % 2
    S = oracle.score(b)["S64"]
    for params in ({}, {"expand_fused": 0}):
        got = M.run(program, b, op=("score", "mine")[seed // 3], prec=prec, params=params)["S"]
        assert np.abs(got.astype(np.float64) - S).max(initial=0.0) <= (2e-2 if prec else 1e-5)


@pytest.mark.parametrize("n,m", [([5, 70], [0, 20]), ([3], [0]), ([130, 0, 64], [1, 9, 300])])
def test_dense_backward_in_bounds(program, n, m):
    # pairs with an empty side; one column; lengths past a row tile
    rng = np.random.default_rng([43, len(n)])
    b = _batch(n, m, 50, [4, 0, 9], [1, 0, 12], seed=5)
    cells = int(np.dot(n, m))
    S, S_raw, E = rng.random(cells), rng.random(cells), rng.standard_normal(cells)
    S, S_raw, E = (x.astype(np.float32) for x in (S, S_raw, E))
    got = M.run(program, b, op="backward", E=E, S=S, S_raw=S_raw)
    np.testing.assert_array_equal(_bits(got["S"]), _bits(E))   # (the gradient of S)
    o = oracle.score(b)
    e, s = E.astype(np.float64), S.astype(np.float64)
    dz = e * s * (1.0 - s)
    ref = np.array([(dz * S_raw).sum(), (dz * o["rho"]).sum(), dz.sum()])
    # FP32 sums of at most `cells` terms, each below 2^-2 * |E|
    tol = 2.0 ** -24 * (64 + np.ceil(cells / 256)) * np.abs(e).sum() / 4
    assert np.abs(got["grad_wb"] - ref).max() <= tol


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("m", [130, 600])   # a workgroup or a wave per tile
def test_values_that_are_not_finite_stay_in_their_cells(program, prec, m):
    """A dictionary value that is infinite, NaN or (BF16) rounds to infinity
    reaches the cells whose source sentence brings it and whose target sentence
    holds its word, and no other."""
    import dataclasses
    b = _batch([21], [m], 300, [3, 1, 0, 12, 40], [5, 33, 0, 70], seed=6)
    bad = np.arange(0, len(b.d_val), 37)
    val = b.d_val.copy()
    val[bad] = np.resize(np.array([np.inf, 3.4e38, np.nan, -np.inf, -3.4e38], np.float32), len(bad))
    if prec == 0:
        val[np.abs(val) == np.float32(3.4e38)] = np.inf
    zero = b.d_val.copy()
    zero[bad] = 0.0
    got = M.run(program, dataclasses.replace(b, d_val=val), prec=prec)
    fin = M.run(program, dataclasses.replace(b, d_val=zero), prec=prec)
    # merged rows in FP64, rounded to FP32; which are not finite as operands
    T = np.zeros((21, b.V))
    with np.errstate(invalid="ignore", over="ignore"):
        for i in range(21):
            for t in b.src_tok[b.src_off[i]:b.src_off[i + 1]]:
                e = slice(b.d_row_off[t], b.d_row_off[t + 1])
                np.add.at(T[i], b.d_col[e], val[e].astype(np.float64))
        T = T.astype(np.float32)
        if prec == 1:
            T[np.abs(T) > 3.3895e38] *= np.float32(10.0)   # (rounds up to infinity)
        ls, lt = np.diff(b.src_off), np.diff(b.tgt_off)
        hit = np.zeros((21, m), bool)
        dot = np.zeros((21, m))
        for j in range(m):
            u = np.unique(b.tgt_tok[b.tgt_off[j]:b.tgt_off[j + 1]])
            odd = ~np.isfinite(T[:, u])
            hit[:, j] = odd.any(1)
            dot[:, j] = np.where(odd, T[:, u], 0.0).sum(1)
        hi, lo = np.maximum(ls[:, None], lt), np.minimum(ls[:, None], lt)
        rho = np.where(hi > 0, lo / np.maximum(hi, 1), 1.0)
        z = b.scorer[0] * dot + b.scorer[1] * rho + b.scorer[2]
        S = 1.0 / (1.0 + np.exp(-z))
    assert hit.any() and not hit.all()
    raw, s = got["S_raw"].reshape(21, m), got["S"].reshape(21, m)
    np.testing.assert_array_equal(raw[hit], dot[hit].astype(np.float32))
    np.testing.assert_array_equal(s[hit], S[hit].astype(np.float32))
    np.testing.assert_array_equal(_bits(raw[~hit]), _bits(fin["S_raw"].reshape(21, m)[~hit]))
    np.testing.assert_array_equal(_bits(s[~hit]), _bits(fin["S"].reshape(21, m)[~hit]))


def _path_case(n, m, cells, rng):
    """Similarities whose best path goes through the given cells."""
    S = (rng.integers(0, 3, (n, m)) / 8.0).astype(np.float32)
    for i, j in cells:
        S[i, j] += 0.75
    return S.ravel()


def _diagonal(i, j, k):
    return [(i + x, j + x) for x in range(k)]


# paths of pairs walked by all their strips at once: on the line from corner to
# corner, a preface or an appendix without a counterpart on either side, along a
# side, in steps, and far to the left within one strip
PATHS = {
    "line": (640, 660, _diagonal(0, 0, 640)),
    "preface": (1100, 500, _diagonal(600, 0, 500)),
    "appendix": (1100, 500, _diagonal(0, 0, 500)),
    "target preface": (560, 1400, _diagonal(0, 840, 560)),
    "target appendix": (560, 1400, _diagonal(0, 0, 560)),
    "side": (1500, 210, _diagonal(0, 0, 210)),
    "steps": (1200, 1200, _diagonal(0, 0, 150) + _diagonal(150, 600, 300) + _diagonal(900, 900, 300)),
    "left": (900, 3000, _diagonal(0, 0, 450) + _diagonal(450, 2550, 450)),
    "narrow": (700, 3, _diagonal(300, 0, 3)),
}


@pytest.mark.parametrize("pairs", [1, 7])   # sixteen or eight strips climbed ahead
def test_traceback_in_bounds(program, pairs):
    rng = np.random.default_rng(47)
    names = sorted(PATHS) if pairs > 1 else ["preface"]
    ns = [PATHS[k][0] for k in names] + [70, 0, 5]
    ms = [PATHS[k][1] for k in names] + [50, 9, 0]
    S = np.concatenate([_path_case(*PATHS[k], rng) for k in names] + [rng.random(70 * 50).astype(np.float32)])
    b = _batch(ns, ms, 10, [0], [0])
    for threshold in (0.5, -1e30):
        got = M.run(program, b, op="align", S=S, gap=-0.125, threshold=threshold, passes=2, order=3 if threshold < 0 else None)
        ora = oracle.align(ns, ms, S, -0.125, threshold)
        H.assert_align_equal(got, ora, ns, ms, check_path_as_kept=threshold < 0)


@pytest.mark.parametrize("tokens,deg", [(48, 8), (49, 2), (49, 3), (80, 4), (80, 5), (81, 2), (81, 3), (81, 4), (128, 6),
                                        (128, 8), (129, 3), (146, 7)])
def test_merge_kinds_in_bounds(program, tokens, deg):
    import dataclasses
    rng = np.random.default_rng([67, tokens, deg])
    V = 600
    b = _batch([9], [40], V, [tokens, 1, 0, tokens // 2], [12, 30, 1], seed=8)
    val = rng.random(V * deg).astype(np.float32)
    b = dataclasses.replace(b, d_row_off=(np.arange(V + 1) * deg).astype(np.int32), d_val=val, d_deg=deg,
                            d_col=rng.integers(0, V, V * deg).astype(np.int32))
    got = M.run(program, b, params={"expand_fused": 0}, apart=True)
    assert got["launches"]["merge"] > 0
    assert H.s_rel_err(got["S"], oracle.score(b)["S64"]).max() <= 1e-5


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("case", ["lengths", "repeats", "row", "table"])
def test_chosen_contractions_in_bounds(program, case, prec):
    b = CASES[case]()
    S = oracle.score(b)["S64"]
    for params in ({"score_kind": 1}, {"score_kind": 1, "expand_fused": 0, "score_kgroup": 2}, {"score_kind": 2}):
        got = M.run(program, b, prec=prec, params=params)["S"]
        assert np.abs(got.astype(np.float64) - S).max() <= (2e-2 if prec else 1e-5)
