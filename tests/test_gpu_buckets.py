"""The refresh of cells that several neurons share at the finest depth: two neurons to thousands,
across the ends of waves and chunks, with and without vacant elements, aggregates against
the oracle bitwise; negative counts in one; trees of few neurons and many nodes. And
its time where 64 neurons share each cell, against as many apart (a member at a time: 2.6
times)."""
import time

import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T, say
from oracle import oracle as orc

pytestmark = pytest.mark.gpu
EDGE = 1000.0


def _cells(rng, sizes):
    pos = np.repeat(rng.uniform(0.0, EDGE, (len(sizes), 3)), sizes, axis=0)
    # the members' own positions differ within the cell
    pos += rng.uniform(0.0, 1e-9, pos.shape)
    return pos[rng.permutation(len(pos))]


def _check(pos, rng):
    n = len(pos)
    t = orc.OracleTree(pos, np.zeros(3), EDGE)
    tree = msp.build_octree(T(pos, torch.float64), np.zeros(3), EDGE)
    assert tree.num_nodes == t.num_nodes
    for _ in range(2):
        ve = rng.integers(0, 4, n).astype(np.int32) * (rng.random(n) < 0.5)
        vi = rng.integers(0, 3, n).astype(np.int32) * (rng.random(n) < 0.1)
        t.update_counts(ve, vi)
        msp.update_vacant_counts(tree, T(ve, torch.int32), T(vi, torch.int32))
        for ty in (0, 1):
            v, c = (x.cpu().numpy() for x in tree.export_aggregates(ty))
            ov, oc = t.aggregates(ty)
            assert np.array_equal(v, ov)
            assert np.array_equal(c[ov > 0].view(np.uint64), oc[ov > 0].view(np.uint64))
    assert tree.last_device_error() == 0
    return tree


@pytest.mark.parametrize("size", [2, 3, 63, 64, 65, 128, 1000, 1024, 5000])
@pytest.mark.parametrize("n", [1500, 4096, 9001, 140000])
def test_cells_of_one_size(size, n):
    rng = np.random.default_rng(size)
    _check(_cells(rng, np.full(max(1, n // size), size))[:n], rng).free()


@pytest.mark.parametrize("seed", range(3))
def test_cells_of_all_sizes(seed):
    rng = np.random.default_rng(seed)
    sizes = rng.choice([1, 2, 5, 63, 64, 65, 129, 700], 500, p=[.4, .2, .2, .05, .05, .05, .03, .02])
    tree = _check(_cells(rng, sizes), rng)
    ve = np.ones(tree.n, np.int32)
    ve[tree.n // 2] = -1
    msp.update_vacant_counts(tree, T(ve, torch.int32), T(ve, torch.int32))
    assert tree.last_device_error() != 0
    tree.free()


def _refresh_time(pos):
    n = len(pos)
    tree = msp.build_octree(T(pos, torch.float64), np.zeros(3), EDGE)
    v = T(np.arange(n) % 3, torch.int32)
    times = []
    for _ in range(8):
        torch.cuda.synchronize()
        t = time.perf_counter()
        msp.update_vacant_counts(tree, v, v)
        torch.cuda.synchronize()
        times.append(time.perf_counter() - t)
    tree.free()
    return min(times[1:])


def test_time_of_cells_of_64():
    n = 1 << 21
    rng = np.random.default_rng(4)
    apart = _refresh_time(rng.uniform(0.0, EDGE, (n, 3)))
    cells = _refresh_time(_cells(rng, np.full(n // 64, 64)))
    say(f"refresh {apart * 1e6:.0f} us, 64 neurons to a cell {cells * 1e6:.0f} us")
    assert cells < 2.0 * apart
