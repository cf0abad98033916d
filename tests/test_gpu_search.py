"""The random search's similarity counted on the GPU against the same counts on
the host, and reference alignments that only the host counts (a source sentence
named twice, a pair outside its documents)."""
import numpy as np
import pytest

from synth import corpus

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["plain", "unordered", "empty", "twice", "outside"])
def test_random_search_similarity(kind):
    import paper_1512_01641_amd as nw
    from paper_1512_01641_amd import tune
    b = corpus.make_batch(3, pairs=5, sizes=([30, 0, 70, 12, 1], [40, 9, 66, 0, 1]))
    off, gold = b.gold_off.copy(), b.gold.copy()
    if kind == "unordered":
        for k in range(b.B):
            gold[off[k]:off[k + 1]] = gold[off[k]:off[k + 1]][::-1].copy()
    elif kind == "empty":
        off, gold = np.zeros(b.B + 1, np.int64), np.zeros((0, 2), np.int32)
    elif kind == "twice":
        gold[1, 0] = gold[0, 0]
    elif kind == "outside":
        gold[0] = (1000, 3)
    mn = nw.Miner(nw.Context(0), nw.DeviceBatch.from_host(b), nw.DeviceDict.from_host(b), 0)
    assert tune._SharedPairs(mn, off, gold).ok == (kind not in ("twice", "outside"))
    r = tune.random_search(mn, b.scorer, off, gold, trials=6, seed=4)
    ref = [gold[off[k]:off[k + 1]] for k in range(b.B)]
    for th, g, sim in r["history"]:
        mn.align(g, th)
        nk, kept = mn.n_kept[:b.B].cpu().numpy(), mn.kept.cpu().numpy()
        auto = [kept[int(mn.p_off[k]):int(mn.p_off[k]) + int(nk[k])] for k in range(b.B)]
        assert sim == tune.similarity(auto, ref)
