"""The alignment fill at the edges of its tiling: 16-step chunks, 64-step
blocks, 64-row strips handed on through LDS row rings of 512 columns and, every
fourth strip, through memory."""
import numpy as np
import pytest

import oracle
from tests import helpers as H

pytestmark = pytest.mark.gpu

SIZES = {
    # three strips; the last column leaves a strip in each step of a chunk, in
    # the first and the last block
    "columns": [(130, m) for m in (1, 2, 15, 16, 17, 18, 47, 48, 49, 63, 64, 65, 66, 81, 127, 128, 129)],
    # one strip, from one row to 64
    "rows": [(n, 70) for n in (1, 2, 15, 16, 17, 63, 64)] + [(64, m) for m in (1, 15, 16, 17, 64, 65)],
    # rows longer than the ring, over three tasks
    "ring": [(520, 1100), (520, 513), (257, 512), (129, 1025), (64, 1500)],
    # strips of several pairs in one task, each with its row from memory
    "memory": [(300, 90)] * 6 + [(370, 20)] * 3 + [(3, 4)] * 2,
}


@pytest.mark.parametrize("staging", [0, 2])
@pytest.mark.parametrize("g", [-0.25, -0.0])
@pytest.mark.parametrize("kind", list(SIZES))
def test_fill_edges_bitexact(kind, g, staging):
    rng = np.random.default_rng(11)
    ns, ms = [a for a, _ in SIZES[kind]], [b for _, b in SIZES[kind]]
    total = sum(a * b for a, b in SIZES[kind])
    # coarse values: exact ties between the three moves
    S = (rng.integers(0, 5, total) / 4.0 - 0.25).astype(np.float32)
    ora = oracle.align(ns, ms, S, g, -1e30)
    gpu = H.gpu_align_only(ns, ms, S, g, -1e30, params={"fill_staging": staging})
    H.assert_align_equal(gpu, ora, ns, ms, check_path_as_kept=True)


def test_fill_infinite_similarities():
    # sums that overflow: a maximum of +-inf still takes UP before LEFT before DIAG
    rng = np.random.default_rng(12)
    sizes = [(40, 50), (130, 70), (300, 300)]
    ns, ms = [a for a, _ in sizes], [b for _, b in sizes]
    S = rng.random(sum(a * b for a, b in sizes)).astype(np.float32)
    hit = rng.random(S.size) < 0.05
    S[hit] = rng.choice(np.array([np.inf, -np.inf, 3e38, -3e38], np.float32), int(hit.sum()))
    ora = oracle.align(ns, ms, S, -0.25, -1e30)
    gpu = H.gpu_align_only(ns, ms, S, -0.25, -1e30)
    H.assert_align_equal(gpu, ora, ns, ms, check_path_as_kept=True)


@pytest.mark.parametrize("n,m,shift", [(193, 60, 0), (256, 4, 0), (257, 1, 0), (300, 900, 500), (900, 300, -500),
                                       (640, 640, 250), (640, 640, -250), (1100, 1100, 0), (4100, 40, 0)])
def test_walk_by_strips_bitexact(n, m, shift):
    """Paths of pairs walked by all their strips at once: along the diagonal,
    far off it (entries no strip's map holds), along a side, and from column 0;
    beside them a pair walked by one wave."""
    rng = np.random.default_rng(13)
    S = (rng.integers(0, 3, (n, m)) / 8.0).astype(np.float32)
    i = np.arange(n)
    j = i + shift
    ok = (j >= 0) & (j < m)
    S[i[ok], j[ok]] += 0.75
    small = rng.random(70 * 50).astype(np.float32)
    flat = np.concatenate([S.ravel(), small])
    ora = oracle.align([n, 70], [m, 50], flat, -0.125, 0.5)
    gpu = H.gpu_align_only([n, 70], [m, 50], flat, -0.125, 0.5)
    H.assert_align_equal(gpu, ora, [n, 70], [m, 50])
    np.testing.assert_array_equal(gpu["n_diag"], ora["n_diag"])
    every = H.gpu_align_only([n, 70], [m, 50], flat, -0.125, -1e30)   # kept = the whole path
    H.assert_align_equal(every, oracle.align([n, 70], [m, 50], flat, -0.125, -1e30), [n, 70], [m, 50],
                         check_path_as_kept=True)
