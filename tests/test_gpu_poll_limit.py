"""The poll limit of the DP means the same waiting time in every staging of the
fill: a strip that reads the row above from LDS does not give up long before one
that polls it in memory.  Forced from the host (the first strip publishes
nothing); every kernel ends normally."""
import numpy as np
import pytest

from tests import helpers as H

pytestmark = pytest.mark.gpu


def _give_up_ms(staging, limit):
    import torch
    import paper_1512_01641_amd as nw
    n, m = [100], [100]
    S = np.random.default_rng(17).random(n[0] * m[0]).astype(np.float32)
    params = {"fill_staging": staging, "dp_spin_limit": limit, "dp_test_hold": 1}
    g = H.gpu_align_only(n, m, S, -0.25, 0.5, params=params)
    score, n_kept, kept = torch.empty(1, device="cuda"), torch.empty(1, dtype=torch.int32, device="cuda"), \
        torch.empty((100, 2), dtype=torch.int32, device="cuda")
    best = np.inf
    for _ in range(3):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        nw.align_batch(g["plan"], g["S"], -0.25, 0.5, score, g["n_diag_t"], kept, n_kept, g["tb"], g["ws"])
        b.record()
        torch.cuda.synchronize()
        assert nw.align_check(g["plan"], g["ws"]) and np.isnan(score.item()) and n_kept.item() == 0
        best = min(best, a.elapsed_time(b))
    return best


def test_limit_takes_as_long_in_every_staging():
    limit = 4000
    ms = {k: _give_up_ms(k, limit) for k in (0, 1, 2)}
    print("ms until a strip gives up, by staging: %s" % ms, flush=True)
    # staging 1 polls memory, as the limit is meant
    assert ms[0] >= 0.9 * ms[1] and ms[2] >= 0.9 * ms[1]
