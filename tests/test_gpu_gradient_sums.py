"""The adjoint's sums over the lanes of a wave, which go four nodes at a time: few entries (groups
that stay partly filled), a tile with one lane, tiles and lanes past the last, with and
without the own-cell test (theta above 1/2), buckets in between, against the oracle."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T
from oracle import oracle as orc
from synth_inputs import uniform_cube

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,theta,bucket", [(2, 0.3, 0), (3, 0.3, 0), (5, 0.9, 0), (6, 0.3, 3),
                                            (65, 0.3, 0), (65, 0.9, 7), (130, 0.0, 0),
                                            (1000, 0.3, 5), (1000, 0.9, 5), (3001, 0.5, 0)])
def test_gradient_matches_oracle(n, theta, bucket):
    w = uniform_cube(n, 500.0, seed=n)
    w.vac_exc[:] = 1 + np.arange(n) % 3
    w.vac_axon[:] = np.arange(n) % 2
    w.neuron_type[:] = np.arange(n) % 5 == 1
    if bucket:
        w.pos[:bucket] = w.pos[0]
    sigma = 200.0
    t = orc.OracleTree(w.pos, w.box_min, w.box_edge)
    t.update_counts(w.vac_exc, w.vac_inh)
    oZ, _, dX, dS = t.attraction(w.neuron_type, w.vac_axon, sigma, theta)
    tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
    msp.update_vacant_counts(tree, T(w.vac_exc, torch.int32), T(w.vac_inh, torch.int32))
    ty, va = T(w.neuron_type, torch.uint8), T(w.vac_axon, torch.int32)
    Z = msp.attraction_fwd(tree, ty, va, sigma, theta)
    np.testing.assert_allclose(Z.cpu().numpy(), oZ, rtol=1e-5)
    src = Z > 0
    gZ = torch.where(src, 1.0 / torch.where(src, Z, torch.ones_like(Z)), torch.zeros_like(Z))
    dpos, ds = msp.attraction_bwd(tree, ty, va, sigma, theta, gZ)
    err = np.abs(dpos.cpu().numpy() - dX)
    assert np.all(err <= 1e-4 * np.abs(dX) + 1e-5 * np.abs(dX).max())
    assert float(ds.item()) == pytest.approx(dS, rel=1e-5)
    tree.free()
