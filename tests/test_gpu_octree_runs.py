"""The octree's sort where neurons share the leading bits of their keys: runs around the
longest that is ordered in place, runs across the blocks that order them, long runs among
short ones, all neurons in one run; keys and (key, id) order against numpy. And its time where
every neuron shares them with nineteen others, against uniform positions (a thread
per run that inserted its neurons in global memory: 2.8 times)."""
import time

import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T, say
from test_gpu_octree_sort import _check

pytestmark = pytest.mark.gpu
EDGE = 1000.0


def _spots(rng, lengths, one_point):
    at = (rng.permutation(512 ** 2)[:len(lengths), None] // np.array([1, 512, 7]) % 512) / 512.0
    pos = np.repeat(at, lengths, axis=0) * EDGE
    if not one_point:
        pos += rng.uniform(0.0, EDGE / 4096.0, pos.shape)
    return pos[rng.permutation(len(pos))]


@pytest.mark.parametrize("one_point", [False, True])
@pytest.mark.parametrize("per, spots", [(127, 80), (128, 80), (129, 80), (257, 40), (5000, 1),
                                        (20, 3000), (130, 2500)])
def test_runs_of_one_length(per, spots, one_point):
    _check(_spots(np.random.default_rng(per), np.full(spots, per), one_point), EDGE)


@pytest.mark.parametrize("seed", range(3))
def test_runs_of_all_lengths(seed):
    rng = np.random.default_rng(seed)
    lengths = rng.choice([1, 2, 3, 40, 127, 128, 129, 300, 4097], 600,
                         p=[.5, .2, .1, .1, .02, .02, .02, .03, .01])
    pos = _spots(rng, lengths, False)
    pos[::17] = pos[0]
    _check(np.concatenate([pos, rng.uniform(0.0, EDGE, (5000, 3))]), EDGE)


def test_all_in_one_run():
    _check(np.random.default_rng(1).uniform(0.0, EDGE / 2048.0, (50001, 3)), EDGE)


def _build_time(pos):
    p = T(pos, torch.float64)
    times = []
    for _ in range(6):
        torch.cuda.synchronize()
        t = time.perf_counter()
        msp.build_octree(p, [0.0, 0.0, 0.0], EDGE).free()
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    return min(times[1:])


def test_time_of_runs_of_twenty():
    n = 1 << 23
    rng = np.random.default_rng(3)
    pos = rng.uniform(0.0, EDGE, (n, 3))
    plain = _build_time(pos)
    runs = np.repeat(pos[: n // 20 + 1], 20, axis=0)[:n] + rng.uniform(0.0, 1e-4 * EDGE, (n, 3))
    runs = _build_time(np.clip(runs, 0.0, EDGE)[rng.permutation(n)])
    say(f"build {plain * 1e6:.0f} us, in runs of twenty {runs * 1e6:.0f} us")
    assert runs < 2.2 * plain
