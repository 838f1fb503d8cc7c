"""Lists that lie where the kernel's weights end, y = d^2 log2(e) / sigma^2 just below 1075:
a pair of neurons (or a cell of some) whose counts make the products positive although
2^-y alone rounds to 0, and networks most of whose sources reach nothing or next to
nothing. What reaches a neuron draws it."""
import numpy as np
import pytest

import paper_2509_26193_amd as msp  # noqa: F401
from gpu_util import compare_search, gpu_search, oracle_tree
from oracle import oracle as orc
from synth_inputs import Workload

pytestmark = pytest.mark.gpu
LOG2E = 1.4426950408889634


def _sigma_for(d2, y):
    """A sigma whose y = d2 * (log2(e) / sigma^2) is at most y and within 2^-28 of it."""
    s = np.sqrt(d2 * LOG2E / y)
    while d2 * (LOG2E / (s * s)) > y:
        s = np.nextafter(s, np.inf)
    assert 0.0 <= y - d2 * (LOG2E / (s * s)) < 2.0 ** -28
    return float(s)


@pytest.mark.parametrize("theta", [0.0, 0.3, 0.9])
@pytest.mark.parametrize("v", [2, 3, 1000])
def test_last_positive_weight(theta, v):
    pos = np.array([[100.0, 100.0, 100.0], [163.0, 116.0, 100.0]])
    sigma = _sigma_for(63.0 ** 2 + 16.0 ** 2, 1075.0 - 2.0 ** -27)
    w = Workload("pair", pos, np.zeros(3), 1000.0, np.zeros(2, np.uint8),
                 np.array([3, 0], np.int32), np.array([0, v], np.int32), np.zeros(2, np.int32),
                 sigma, theta, seed=3)
    g = gpu_search(w)
    # v products of 2^-1074 / 2, added and rounded to a multiple of 2^-1074
    assert np.all(np.abs(g["z0"] - v * 0.5 * 2.0 ** -1074) <= 2.0 ** -1074)
    assert np.all(g["z0"] > 0.0)
    assert np.all(g["target"] == 1)
    g["tree"].free()


@pytest.mark.parametrize("theta", [0.0, 0.3, 0.9])
@pytest.mark.parametrize("n, reach", [(300, 0.7), (300, 1.5), (4000, 0.9), (4000, 1.7)])
def test_sparse_reach_matches_oracle(theta, n, reach):
    """Weights end at `reach` mean distances between neurons."""
    rng = np.random.default_rng(n)
    edge = 1000.0
    sigma = reach * edge / n ** (1.0 / 3.0) / np.sqrt(1075.0 / LOG2E)
    w = Workload("sparse", rng.uniform(0.0, edge, (n, 3)), np.zeros(3), edge,
                 (rng.random(n) < 0.2).astype(np.uint8), rng.integers(0, 3, n).astype(np.int32),
                 rng.integers(0, 4, n).astype(np.int32), rng.integers(0, 4, n).astype(np.int32),
                 sigma, theta, seed=8)
    g = gpu_search(w)
    _, src, elem = orc.search_list(w.vac_axon)
    o = oracle_tree(w).find_targets(w.neuron_type, sigma, theta, w.seed, w.step, src, elem)
    normal = (o["z0"] > 2.0 ** -1000) | (o["z0"] == 0.0)
    assert np.any(o["z0"] > 0.0) and (np.any(o["z0"] == 0.0) or reach > 1.0)
    compare_search(g["target"][normal], g["z0"][normal], {k: o[k][normal] for k in
                                                           ("target", "z0", "window")})
    g["tree"].free()
