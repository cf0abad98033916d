"""The traceback by strips where the path is off the maps: bit for bit against
the oracle, and in about the time of a path on them."""
import numpy as np
import pytest

import oracle
from tests import helpers as H
from tests.test_host_kernels import PATHS, _diagonal, _path_case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", sorted(PATHS))
def test_paths_off_the_maps_bitexact(name):
    n, m, cells = PATHS[name]
    S = _path_case(n, m, cells, np.random.default_rng(53))
    for threshold in (0.5, -1e30):
        gpu = H.gpu_align_only([n], [m], S, -0.125, threshold)
        H.assert_align_equal(gpu, oracle.align([n], [m], S, -0.125, threshold), [n], [m],
                             check_path_as_kept=threshold < 0)


def test_many_pairs_off_the_maps_bitexact():
    # more pairs than compute units: fewer waves climb ahead for each
    n, pairs = 520, 300
    rng = np.random.default_rng(59)
    one = [_path_case(n, n, _diagonal(0, d, n - d), rng) for d in (0, 200, 260, 330)]
    S = np.concatenate([one[k % 4] for k in range(pairs)])
    gpu = H.gpu_align_only([n] * pairs, [n] * pairs, S, -0.125, 0.5)
    H.assert_align_equal(gpu, oracle.align([n] * pairs, [n] * pairs, S, -0.125, 0.5), [n] * pairs, [n] * pairs)


def _walk_us(n, m, cells):
    import torch
    import paper_1512_01641_amd as nw
    S = _path_case(n, m, cells, np.random.default_rng(61))
    g = H.gpu_align_only([n], [m], S, -0.125, 0.5)
    kept = torch.empty((min(n, m), 2), dtype=torch.int32, device="cuda")
    out = [torch.empty(1, dtype=t, device="cuda") for t in (torch.float32, torch.int32, torch.int32)]
    g["plan"].set_timing(True)
    us = []
    for _ in range(6):
        nw.align_batch(g["plan"], g["S"], -0.125, 0.5, out[0], out[1], kept, out[2], g["tb"], g["ws"])
        torch.cuda.synchronize()
        us.append(1000.0 * g["plan"].kernel_ms()["walk"][0])
    return min(us[1:])


def test_paths_off_the_maps_take_no_multiple_of_the_time():
    on = _walk_us(4096, 2560, [(i, i * 2560 // 4096) for i in range(0, 4096, 2)])
    off = {k: _walk_us(4096, 2560, c) for k, c in (("preface", _diagonal(1536, 0, 2560)),
                                                   ("appendix", _diagonal(0, 0, 2560)))}
    print("traceback of 4096 x 2560, us: on the line %.0f, off it %s" % (on, off), flush=True)
    # climbed one strip after another it takes seven times as long
    assert max(off.values()) < 4.0 * on
