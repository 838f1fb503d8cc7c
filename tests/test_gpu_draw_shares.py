"""The draws by shares of a source's elements (launches of up to 16 384 tiles) and by groups of
blocks per die (from 256 blocks of 4 tiles on): no sources at all, one, sizes around a whole
group, and a launch of more tiles than that against two of fewer."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T, compare_search
from oracle import oracle as orc
from synth_inputs import uniform_cube

pytestmark = pytest.mark.gpu


def _find(tree, w, va, theta):
    tgt, off = msp.find_targets(tree, T(w.neuron_type, torch.uint8), T(va, torch.int32), w.sigma,
                                theta, w.seed, w.step)[:2]
    torch.cuda.synchronize()
    return tgt.cpu().numpy(), off.cpu().numpy()


@pytest.mark.parametrize("n,sources", [(50, 0), (50, 1), (3000, 2999), (66000, 65280), (66000, 65536),
                                       (66000, 65600)])
def test_targets_match_oracle(n, sources):
    w = uniform_cube(n, 200.0 * n ** (1.0 / 3.0), seed=sources % 83 + 1)
    rng = np.random.default_rng(n + sources)
    w.vac_axon[:] = 0
    w.vac_axon[rng.permutation(n)[:sources]] = 1 + np.arange(sources) % 5
    t = orc.OracleTree(w.pos, w.box_min, w.box_edge)
    t.update_counts(w.vac_exc, w.vac_inh)
    off, src, elem = orc.search_list(w.vac_axon)
    o = t.find_targets(w.neuron_type, w.sigma, 0.5, w.seed, w.step, src, elem)
    tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
    msp.update_vacant_counts(tree, T(w.vac_exc, torch.int32), T(w.vac_inh, torch.int32))
    tgt, o2 = _find(tree, w, w.vac_axon, 0.5)
    assert np.array_equal(o2, off)
    tgt = tgt[:off[-1]]
    dt, _, z0 = msp.find_targets(tree, T(w.neuron_type, torch.uint8), T(w.vac_axon, torch.int32),
                                 w.sigma, 0.5, w.seed, w.step, diag=True)[:3]
    assert np.array_equal(dt.cpu().numpy()[:off[-1]], tgt)
    if sources:
        compare_search(tgt.astype(np.int64), z0.cpu().numpy(), o, f"{n} {sources}")
    tree.free()


def test_many_tiles_equal_two_halves():
    n = 1100000
    w = uniform_cube(n, 200.0 * n ** (1.0 / 3.0), seed=5)
    w.vac_axon[:] = 1 + np.arange(n) % 3                # 17 188 tiles
    tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
    msp.update_vacant_counts(tree, T(w.vac_exc, torch.int32), T(w.vac_inh, torch.int32))
    tgt, off = _find(tree, w, w.vac_axon, 0.5)
    for half in (0, 1):
        mine = np.arange(n) // 64 % 2 == half
        t2, o2 = _find(tree, w, np.where(mine, w.vac_axon, 0), 0.5)
        e = np.repeat(mine, np.diff(off))
        assert o2[-1] == e.sum()
        assert np.array_equal(t2[:o2[-1]], tgt[:off[-1]][e])
    tree.free()
