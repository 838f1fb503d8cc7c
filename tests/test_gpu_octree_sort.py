"""The octree's sort at the edges of its variants (one block up to 4 096 neurons; blocks that
add up their own offsets up to 64 tiles of 4 096; scanned histograms beyond) and where many
neurons share the leading key bits: sorted keys and (key, id) order against numpy."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T

pytestmark = pytest.mark.gpu


def _keys(pos, edge):
    q = np.clip(np.floor(pos / edge * 2097152.0), 0, 2097151).astype(np.uint64)
    out = np.zeros(len(pos), np.uint64)
    for b in range(21):
        for a in range(3):
            out |= ((q[:, a] >> np.uint64(b)) & np.uint64(1)) << np.uint64(3 * b + 2 - a)
    return out


def _check(pos, edge):
    tree = msp.build_octree(T(pos, torch.float64), [0.0, 0.0, 0.0], edge)
    topo = tree.export_topology()
    k = _keys(pos, edge)
    order = np.argsort(k, kind="stable")
    assert np.array_equal(topo["keys"].cpu().numpy().view(np.uint64), k[order])
    assert np.array_equal(topo["order"].cpu().numpy(), order)
    tree.free()


@pytest.mark.parametrize("n", [1, 2, 63, 65, 255, 1025, 4095, 4096, 4097, 8193, 60001, 262143,
                               262144, 262145, 500003])
def test_uniform(n):
    _check(np.random.default_rng(n).uniform(0.0, 1000.0, (n, 3)), 1000.0)


# neurons per spot that share their leading 32 bits: none sorted by runs, the longest run
# that is, the shortest that is not, many; spread within the spot or on one point
@pytest.mark.parametrize("per", [2, 24, 25, 300])
@pytest.mark.parametrize("one_point", [False, True])
@pytest.mark.parametrize("spots", [3, 700])
def test_shared_leading_bits(per, one_point, spots):
    rng = np.random.default_rng(per + spots)
    # spots on a grid of 2^-9 of the edge, neurons within 2^-12 of it
    at = (rng.permutation(512 ** 2)[:spots, None] // np.array([1, 512, 7]) % 512) / 512.0
    pos = np.repeat(at, per, axis=0) * 1000.0
    if not one_point:
        pos += rng.uniform(0.0, 1000.0 / 4096.0, pos.shape)
    _check(pos[rng.permutation(len(pos))], 1000.0)
