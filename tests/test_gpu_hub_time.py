"""A neuron that owns a large share of the synapses is retracted by many blocks: a step over 2 M
synapses, a third of them one source's, takes a small multiple of the step over the same
list without it (one block and its serial additions: 64 times)."""
import time

import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T, say

pytestmark = pytest.mark.gpu


def _step_time(n, m, share):
    rng = np.random.default_rng(2)
    src, tgt = rng.integers(0, n, m), rng.integers(0, n, m)
    src[rng.random(m) < share] = 3
    ty = src % 5 == 4
    bound = np.zeros((3, n), np.int64)
    np.add.at(bound[0], src, 1)
    for k in (0, 1):
        np.add.at(bound[1 + k], tgt[ty == k], 1)
    z = np.maximum(bound - (rng.random(bound.shape) < 0.1) + 0.5, 0.0)
    z[0, 3] = bound[0, 3] * 0.6
    zero = T(np.zeros(n), torch.int32)
    d = msp.Network(zero, zero, zero, capacity=m)
    saved = [T(a, t.dtype) for a, t in ((z, d.z), (bound, d.bound), (src, d.src), (tgt, d.tgt),
                                        (ty, d.type))]
    times = []
    for _ in range(6):
        for x, y in zip((d.z, d.bound, d.src, d.tgt, d.type), saved):
            x.copy_(y)
        d.m = m
        torch.cuda.synchronize()
        t = time.perf_counter()
        d.step(9, 0, dict(growth_rate=0.0, delete_fraction=0.02))
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    assert np.all(d.bound.cpu().numpy() <= np.floor(z))
    return min(times[1:])


def test_one_owner_of_a_third():
    plain, hub = (_step_time(100_000, 2_000_000, s) for s in (0.0, 0.33))
    say(f"step {plain * 1e6:.0f} us, with one owner of a third {hub * 1e6:.0f} us")
    assert hub < 16.0 * plain
