"""Synapses in the list that bind nothing (an endpoint outside [0, n) or a type above 1:
msp_plasticity_record appends them and reports them) are nobody's to retract, and their
deletion frees nothing."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T

pytestmark = pytest.mark.gpu
N = 8


def _network(seed):
    """Three bound synapses of each neuron among many that bind nothing; neuron 7 has one
    element of each kind too many, the others none."""
    rng = np.random.default_rng(seed)
    ok = [(i, (3 * i + 2 * k + 1) % N, k % 2) for i in range(N) for k in range(3)]
    bad = [(i, g, t) for i, g, t in
           ((7, -1, 0), (7, -1, 1), (7, N, 0), (7, N, 1), (-1, 7, 0), (-1, 7, 1), (N, 7, 0),
            (N, 7, 1), (7, 7, 2), (7, -N, 1), (7, -N - 1, 1), (7, 2 * N - 1, 0))]
    rows = np.array(ok + bad * 20)
    rows = rows[rng.permutation(len(rows))]
    src, tgt, ty = rows.T
    valid = (src >= 0) & (src < N) & (tgt >= 0) & (tgt < N) & (ty <= 1)
    bound = np.zeros((3, N), np.int32)
    np.add.at(bound[0], src[valid], 1)
    np.add.at(bound, (1 + ty[valid], tgt[valid]), 1)
    return src, tgt, ty, valid, bound


def _on_device(src, tgt, ty, bound, z):
    m = src.size
    zero = T(np.zeros(N), torch.int32)
    d = msp.Network(zero, zero, zero, capacity=m)
    # the bound counts lie between rows that nothing may change
    rows = T(np.concatenate([np.full((1, N), 99), bound, np.full((1, N), 99)]), torch.int32)
    d.bound = rows[1:4]
    d.z.copy_(torch.as_tensor(z))
    for x, y in ((d.src, src), (d.tgt, tgt), (d.type, ty)):
        x[:m].copy_(torch.as_tensor(y))
    d.m = m
    return d, rows


@pytest.mark.parametrize("seed", range(4))
def test_only_bound_synapses_are_retracted(seed):
    src, tgt, ty, valid, bound = _network(seed)
    z = bound + 0.5
    z[:, 7] -= (bound[:, 7] > 0)
    d, rows = _on_device(src, tgt, ty, bound, z)
    d.step(4, 1, dict(growth_rate=0.0, delete_fraction=0.0))
    s, g, t = (x.cpu().numpy().astype(np.int64) for x in d.synapses())
    left = (s >= 0) & (s < N) & (g >= 0) & (g < N) & (t <= 1)
    assert int((~left).sum()) == int((~valid).sum())
    after = np.zeros((3, N), np.int32)
    np.add.at(after[0], s[left], 1)
    np.add.at(after, (1 + t[left], g[left]), 1)
    assert np.array_equal(d.bound.cpu().numpy(), after)
    assert np.all(after <= np.floor(z))
    assert 1 <= int(valid.sum() - left.sum()) <= 3
    assert torch.all(rows[[0, 4]] == 99)


def test_deletion_frees_bound_elements_only():
    src, tgt, ty, _, bound = _network(9)
    d, rows = _on_device(src, tgt, ty, bound, bound + 0.5)
    d.step(4, 1, dict(growth_rate=0.0, delete_fraction=1.0))
    assert d.m == 0
    assert torch.all(d.bound == 0)
    assert torch.all(rows[[0, 4]] == 99)
