"""Deletion and retraction where their selections change form: lists around the 4 096
synapses up to which every priority is kept, and neurons with none, a few, 64, 65 and most
of the synapses to retract from. Element counts do not grow here; everything integer
equals the oracle's."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T
from oracle import oracle as orc

pytestmark = pytest.mark.gpu


def _network(n, m, seed):
    """A list with hubs (neuron 3 a source, 5 a target of a third of it each, 7 and 8 of
    exactly 64 and 65 synapses) and element counts that leave every kind of excess."""
    rng = np.random.default_rng(seed)
    src = rng.integers(0, n, m).astype(np.int32)
    tgt = rng.integers(0, n, m).astype(np.int32)
    src[rng.random(m) < 0.33] = 3
    tgt[rng.random(m) < 0.33] = 5
    for hub, k in ((7, 64), (8, 65)):
        src[src == hub] = 9
        src[rng.permutation(m)[:min(k, m)]] = hub
    ty = (src % 5 == 4).astype(np.uint8)
    bound = np.zeros((3, n), np.int32)
    np.add.at(bound[0], src, 1)
    for k in (0, 1):
        np.add.at(bound[1 + k], tgt[ty == k], 1)
    z = bound + rng.integers(-3, 3, bound.shape) + 0.5
    z[0, [3, 7, 8]] = bound[0, [3, 7, 8]] * 0.4 + 0.25
    z[:, 5] = bound[:, 5] * 0.7
    z[0, 11] = 0.0
    return src, tgt, ty, np.maximum(z, 0.0), bound


@pytest.mark.parametrize("m", [1, 70, 4095, 4096, 4097, 20000, 300001])
@pytest.mark.parametrize("frac", [0.0, 0.1, 0.5, 1.0])
def test_step_matches_oracle(m, frac):
    n = 300
    src, tgt, ty, z, bound = _network(n, m, seed=m)
    zero = np.zeros(n, np.int32)
    d = msp.Network(*(T(zero, torch.int32),) * 3, capacity=m + 5)
    o = orc.Network(zero, zero, zero, capacity=m + 5)
    for x, y in ((d.z, z), (d.bound, bound)):
        x.copy_(torch.as_tensor(y))
    for x, y in ((d.src, src), (d.tgt, tgt), (d.type, ty)):
        x[:m].copy_(torch.as_tensor(y))
    d.m = m
    o.z[:], o.bound[:], o.m = z, bound, m
    o.src[:m], o.tgt[:m], o.type[:m] = src, tgt, ty
    for step in (0, 1):
        dv = d.step(9, step, dict(growth_rate=0.0, delete_fraction=frac))
        ov = o.step(9, step, dict(nu=0.0, delete_frac=frac))
        assert d.m == o.m
        for a, b in zip(d.synapses(), o.synapses()):
            assert np.array_equal(a.cpu().numpy(), b), (m, frac, step)
        assert np.array_equal(d.bound.cpu().numpy(), o.bound)
        for a, b in zip(dv, ov):
            assert np.array_equal(a.cpu().numpy(), b)
