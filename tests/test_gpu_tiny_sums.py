"""Sources whose whole level-0 list lies 24 to 27 kernel widths away: their weights are below
2^-830, and from y = d^2 log2(e) / sigma^2 > 1022 on no longer normal doubles. The sums
and draws there are as exact as elsewhere."""
import math

import numpy as np
import pytest

import paper_2509_26193_amd as msp  # noqa: F401
from gpu_util import gpu_search, oracle_tree
from oracle import oracle as orc
from synth_inputs import Workload

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("y", [850.0, 899.0, 905.0, 1010.0, 1030.0, 1060.0, 1073.5, 1090.0])
@pytest.mark.parametrize("theta", [0.0, 0.3])
def test_far_list(y, theta):
    rng = np.random.default_rng(int(y))
    sigma, ns, nt = 750.0, 70, 40
    d = sigma * math.sqrt(y / 1.4426950408889634)
    pos = np.concatenate([rng.uniform(0.0, 0.02, (ns, 3)),
                          np.array([d, 0.0, 0.0]) + rng.uniform(0.0, 0.02, (nt, 3))])
    n = ns + nt
    ax = np.zeros(n, np.int32)
    ax[:ns] = 2
    v = np.zeros(n, np.int32)
    v[ns:] = rng.integers(1, 4, nt)
    w = Workload("far", pos, np.zeros(3), 25000.0, np.zeros(n, np.uint8), ax, v,
                 np.zeros(n, np.int32), sigma, theta, seed=5)
    g = gpu_search(w)
    _, src, elem = orc.search_list(ax)
    o = oracle_tree(w).find_targets(w.neuron_type, sigma, theta, w.seed, w.step, src, elem)
    # the oracle rounds each exp(-x) to a multiple of 2^-1074 before the product with v, the
    # library the product or the sum of products
    tol = 1e-5 * o["z0"] + (v.sum() + nt) * 2.0 ** -1074
    assert np.all(np.abs(g["z0"] - o["z0"]) <= tol)
    assert np.array_equal(g["z0"] > 0, o["z0"] > 0) or 1074.0 < y < 1076.0
    assert np.all((g["target"] >= ns) == (g["z0"] > 0))
    if y < 1020.0:
        diff = g["target"] != o["target"]
        assert np.all(o["window"][diff] < 1e-6)
    g["tree"].free()
