"""The selection of a key by its rank, as the deletion falls back to it and the retraction of
owners with many candidates uses it (csrc/plasticity.hpp, kth_key and del_pick_k), on keys
that priorities do not make: equal ones, few different ones, all bits and none, lists around
those that are ranked at once; and the deletion's choice where the kept range misses the
wanted rank or a block's room overflowed. Against numpy's order by (key, index)."""
import ctypes
import os

import numpy as np
import pytest
import torch

from gpu_util import DEV

pytestmark = pytest.mark.gpu
NATIVE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "native")


@pytest.fixture(scope="module")
def probe():
    path = os.path.join(NATIVE, "libpick_probe.so")
    if not os.path.exists(path):
        from paper_2509_26193_amd import build_lib
        build_lib.compile_hip(os.path.join(NATIVE, "pick_probe.hip"), path)
    return ctypes.CDLL(path)


def _u64(a):
    return torch.as_tensor(np.ascontiguousarray(a, np.uint64).view(np.int64), device=DEV)


def _p(t):
    return ctypes.c_void_p(t.data_ptr())


def _keys(kind, c, rng):
    if kind == "uniform":
        return rng.integers(0, 1 << 64, c, dtype=np.uint64)
    if kind == "equal":
        return np.full(c, 0xDEADBEEF12345678, np.uint64)
    if kind == "ends":
        return rng.choice(np.array([0, (1 << 64) - 1], np.uint64), c)
    if kind == "low":                       # different in the last four bits alone
        return np.uint64(0xABCDEF0123456780) + rng.integers(0, 16, c).astype(np.uint64)
    if kind == "few":
        return rng.choice(rng.integers(0, 1 << 64, 5, dtype=np.uint64), c)
    return np.uint64(1 << 63) + rng.permutation(c).astype(np.uint64)       # "dense"


@pytest.mark.parametrize("kind", ["uniform", "equal", "ends", "low", "few", "dense"])
@pytest.mark.parametrize("c", [1, 2, 255, 256, 257, 1023, 1025, 5000, 70001])
def test_key_of_rank(probe, kind, c):
    rng = np.random.default_rng(c)
    key = _keys(kind, c, rng)
    order = np.lexsort((np.arange(c), key))
    ranks = np.unique(np.concatenate([[1, c, (c + 1) // 2], rng.integers(1, c + 1, 6)]))
    k, r = _u64(key), torch.as_tensor(ranks, device=DEV)
    for threads in (256, 1024):
        ok, oi = torch.zeros(len(ranks), dtype=torch.int64, device=DEV), \
            torch.full((len(ranks),), -1, dtype=torch.int64, device=DEV)
        assert probe.probe_kth(_p(k), ctypes.c_int64(c), _p(r), len(ranks), threads, _p(ok),
                               _p(oi)) == 0
        assert np.array_equal(oi.cpu().numpy(), order[ranks - 1]), (kind, c, threads)
        assert np.array_equal(ok.cpu().numpy().view(np.uint64), key[order[ranks - 1]])


@pytest.mark.parametrize("kind", ["uniform", "equal", "few"])
@pytest.mark.parametrize("how", ["range above", "range below", "overflow"])
@pytest.mark.parametrize("m", [4097, 30011])
@pytest.mark.parametrize("frac", [0.001, 0.37, 1.0])
def test_deletion_searches_all(probe, kind, how, m, frac):
    rng = np.random.default_rng(m)
    key = _keys(kind, m, rng)
    want = int(np.floor(frac * m + 0.5))
    blocks, room = 17, probe.probe_del_room()
    below = np.zeros(blocks, np.int64)
    kept = np.zeros(blocks, np.int32)
    if how == "range above":                # the wanted rank lies above what was kept
        below[3] = want - 1 if want > 1 else 0
    elif how == "range below":
        below[5] = want
    else:
        kept[2] = room + 1
    k, b, n = _u64(key), torch.as_tensor(below, device=DEV), torch.as_tensor(kept, device=DEV)
    ck = torch.zeros(blocks * room, dtype=torch.int64, device=DEV)
    ci = torch.zeros(blocks * room, dtype=torch.int32, device=DEV)
    st = torch.zeros(2, dtype=torch.int64, device=DEV)
    assert probe.probe_del_pick(ctypes.c_double(frac), ctypes.c_int64(m), blocks, _p(k), _p(b),
                                _p(n), _p(ck), _p(ci), _p(st)) == 0
    order = np.lexsort((np.arange(m), key))
    got = st.cpu().numpy()
    assert got[1] == order[want - 1]
    assert got.view(np.uint64)[0] == key[order[want - 1]]
