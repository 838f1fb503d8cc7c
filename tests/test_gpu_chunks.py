"""The refresh and the adjoint's push-down by chunks of the tree, at the sizes where their form
changes (one chunk up to 4 096 neurons, one run of chunks up to 131 072, several beyond;
both types' counts side by side from 262 145 on),
with single neurons, coincident ones across chunk ends and deep chains: topology and
aggregates against the oracle bitwise, a second refresh included."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T
from oracle import oracle as orc
from synth_inputs import uniform_cube

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,form", [(1, ""), (2, ""), (1023, "chain"), (4096, ""), (4097, ""),
                                    (4097, "coincident"), (5121, "chain"), (20000, "coincident"),
                                    (131072, ""), (131073, ""), (262144, ""),
                                    (262145, "coincident"), (1200000, "coincident")])
def test_refresh_matches_oracle(n, form):
    w = uniform_cube(n, 3000.0, seed=n % 97)
    rng = np.random.default_rng(n)
    if form == "coincident":                # groups of 2 to 3000 neurons on one point
        at = 0
        for k in (2, 3, 64, 300, 900, 3000):
            w.pos[at:at + k] = w.pos[at]
            at += k + 7
    if form == "chain":                     # pairs a finest cell apart, and a nested sequence
        w.pos[1:800:2] = w.pos[0:799:2] + 3000.0 / 2097152.0
        w.pos[800:820] = 1500.0 * 2.0 ** -np.arange(20)[:, None]
    w.pos = w.pos[rng.permutation(n)]
    t = orc.OracleTree(w.pos, w.box_min, w.box_edge)
    tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
    nd, topo = t.nodes(), tree.export_topology()
    assert tree.num_nodes == t.num_nodes
    for a, b in (("depth", "depth"), ("begin", "begin"), ("end", "end"),
                 ("subtree_end", "subtree_end")):
        assert np.array_equal(topo[a].cpu().numpy(), nd[b]), a
    for k in range(2):
        ve = rng.integers(0, 4, n).astype(np.int32) * (rng.random(n) < 0.6)
        vi = rng.integers(0, 3, n).astype(np.int32)
        t.update_counts(ve, vi)
        msp.update_vacant_counts(tree, T(ve, torch.int32), T(vi, torch.int32))
        for ty in (0, 1):
            v, c = (x.cpu().numpy() for x in tree.export_aggregates(ty))
            ov, oc = t.aggregates(ty)
            assert np.array_equal(v, ov)
            assert np.array_equal(c[ov > 0].view(np.uint64), oc[ov > 0].view(np.uint64))
    assert tree.last_device_error() == 0
    tree.free()


@pytest.mark.parametrize("n", [4096, 4097, 9000])
def test_gradient_with_coincident_neurons(n):
    w = uniform_cube(n, 1300.0, seed=n)
    w.pos[10:310] = w.pos[10]
    tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
    msp.update_vacant_counts(tree, T(w.vac_exc, torch.int32), T(w.vac_inh, torch.int32))
    ty, va = T(w.neuron_type, torch.uint8), T(w.vac_axon, torch.int32)
    Z = msp.attraction_fwd(tree, ty, va, w.sigma, w.theta)
    src = va > 0
    gZ = torch.where(src, 1.0 / torch.where(src, Z, torch.ones_like(Z)), torch.zeros_like(Z))
    dpos, ds = msp.attraction_bwd(tree, ty, va, w.sigma, w.theta, gZ)
    t = orc.OracleTree(w.pos, w.box_min, w.box_edge)
    t.update_counts(w.vac_exc, w.vac_inh)
    _, _, dX, dS = t.attraction(w.neuron_type, w.vac_axon, w.sigma, w.theta)
    err = np.abs(dpos.cpu().numpy() - dX)
    assert np.all(err <= 1e-4 * np.abs(dX) + 1e-5 * np.abs(dX).max())
    assert float(ds.item()) == pytest.approx(dS, rel=1e-5)
    tree.free()
