"""Launches with few tiles cut each tile's level-0 walk into up to 64 parts, at runs of
sorted neurons: the lists, draws and targets are those of the whole walk."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T
from synth_inputs import config_clusters, uniform_cube

pytestmark = pytest.mark.gpu


def _run(tree, w, va, parts):
    ty = T(w.neuron_type, torch.uint8)
    tgt, off, z0, lv, cnt = msp.find_targets(tree, ty, va, w.sigma, w.theta, w.seed, w.step,
                                             diag=True, counters=True, parts=parts)
    torch.cuda.synchronize()
    out = dict(target=tgt.cpu().numpy(), z0=z0.cpu().numpy(), levels=lv.cpu().numpy())
    out.update({k: v.cpu().numpy() for k, v in cnt.items() if k != "wave_steps"})
    return out


def _case(name):
    if name == "coincident":                  # a bucket leaf of many neurons, and a few more
        w = uniform_cube(700, 500.0, seed=61)
        w.pos[40:240] = w.pos[40]
        return w
    if name == "chain":                       # deep single-child chains
        w = uniform_cube(300, 1000.0, seed=62)
        w.pos[:64] = 1e-3 * w.pos[:64]
        return w
    if name == "clusters":
        return config_clusters(seed=63, n_centres=5, per_centre=1300, edge=8000.0)
    if name == "sparse":                      # few tiles over many runs of neurons
        w = uniform_cube(70001, 2600.0, seed=64)
        keep = np.random.default_rng(65).random(w.n) < 0.01
        w.vac_axon[~keep] = 0
        return w
    n = int(name)
    return uniform_cube(n, 1000.0 * max(1.0, n / 4096.0) ** (1.0 / 3.0), seed=66 + n % 7)


@pytest.mark.parametrize("case", ["1", "2", "9", "65", "513", "4096", "33000", "coincident",
                                  "chain", "clusters", "sparse"])
@pytest.mark.parametrize("theta", [0.0, 0.3, 0.7])
def test_many_parts_equal_whole_walk(case, theta):
    """Few tiles are cut into up to 64 parts at runs of sorted neurons (1, 8 or 64 runs of 8
    neurons, a last run that is not full): the lists and draws are those of the whole walk."""
    w = _case(case)
    if theta == 0.0 and w.n > 5000:
        pytest.skip("the direct sum over many neurons")
    tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
    msp.update_vacant_counts(tree, T(w.vac_exc, torch.int32), T(w.vac_inh, torch.int32))
    va = T(w.vac_axon, torch.int32)
    w.theta = theta
    ref, g = _run(tree, w, va, 1), _run(tree, w, va, 0)
    for k in ("target", "levels", "visits", "opens", "visits0", "opens0", "entries0"):
        assert np.array_equal(g[k], ref[k]), (case, theta, k)
    # the same non-negative terms added in another grouping: each sum of up to 70 000 terms
    # is within 7e4 * 2^-53 of exact
    assert np.all(np.abs(g["z0"] - ref["z0"]) <= 2e-11 * ref["z0"])
    plain, _ = msp.find_targets(tree, T(w.neuron_type, torch.uint8), va, w.sigma, theta, w.seed,
                                w.step)
    assert np.array_equal(plain.cpu().numpy(), ref["target"]), (case, theta)
    tree.free()
