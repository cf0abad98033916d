"""The two-kernel merge at the edges of what it loads ahead: 48, 80 and 128
tokens per sentence and four or eight dictionary entries per word, and tables
filled to the plan's bound by words that all differ."""
import dataclasses

import numpy as np
import pytest

import oracle
from synth import corpus
from tests import helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tokens,deg", [(48, 4), (48, 8), (49, 4), (80, 8), (81, 3), (128, 8), (130, 7), (16, 64), (1, 5)])
def test_merge_kinds(tokens, deg):
    rng = np.random.default_rng([31, tokens, deg])
    V = 5003
    b = corpus.make_batch(2, sizes=([1], [1]), V=V)
    n, m = [20, 3], [70, 1]
    s = np.resize([tokens, 1, 0, tokens // 2, tokens], sum(n))
    t = np.resize([12, 30, 1], sum(m))
    col = (np.arange(V)[:, None] * deg + np.arange(deg)) % V   # neighbouring words share no translation
    b = dataclasses.replace(
        b, n=np.asarray(n, np.int32), m=np.asarray(m, np.int32),
        src_off=np.concatenate([[0], np.cumsum(s)]).astype(np.int64),
        src_tok=np.concatenate([rng.choice(V // deg, k, replace=False) for k in s]).astype(np.int32),
        tgt_off=np.concatenate([[0], np.cumsum(t)]).astype(np.int64),
        tgt_tok=rng.integers(0, V, int(t.sum())).astype(np.int32),
        d_row_off=(np.arange(V + 1) * deg).astype(np.int32), d_col=col.ravel().astype(np.int32),
        d_val=rng.random(V * deg).astype(np.float32), d_deg=deg,
        gold_off=np.zeros(3, np.int64), gold=np.zeros((0, 2), np.int32))
    got = H.run_gpu(b, prec=0, params={"expand_fused": 0})
    assert H.s_rel_err(got["S"], oracle.score(b)["S64"]).max() <= 1e-5
