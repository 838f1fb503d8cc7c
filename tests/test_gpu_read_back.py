"""The values that calls read back through leased page-locked slots: many threads at once on
streams of their own get their own values, a commit of no requests reports none formed, and
bad synapses are still reported by the record, which appends and binds in one launch."""
import threading

import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T
from synth_inputs import uniform_cube

pytestmark = pytest.mark.gpu


def _update(w, stream=None):
    with torch.cuda.stream(stream or torch.cuda.current_stream()):
        ty, va = T(w.neuron_type, torch.uint8), T(w.vac_axon, torch.int32)
        ve, vi = T(w.vac_exc, torch.int32), T(w.vac_inh, torch.int32)
        tree = msp.build_octree(T(w.pos, torch.float64), w.box_min, w.box_edge)
        msp.update_vacant_counts(tree, ve, vi)
        tgt, off = msp.find_targets(tree, ty, va, w.sigma, 0.4, w.seed, 0)[:2]
        syn = msp.commit_synapses(tgt, off, ty, va, ve, vi, w.seed, 0)
        out = [tree.num_nodes, syn["n_formed"], off.cpu().numpy(), tgt.cpu().numpy()]
        out += [syn[k].cpu().numpy() for k in ("syn_src", "syn_tgt", "syn_type")]
        tree.free()
        return out


def test_many_threads_read_their_own_values():
    nets = [uniform_cube(300 + 371 * k, 600.0, seed=k) for k in range(12)]
    want = [_update(w) for w in nets]
    torch.cuda.synchronize()
    got, errors = [None] * len(nets), []

    def work(k):
        try:
            s = torch.cuda.Stream()
            for _ in range(5):
                got[k] = _update(nets[k], s)
                for a, b in zip(got[k], want[k]):
                    assert np.array_equal(a, b), k
        except Exception as e:                     # reported by the main thread
            errors.append((k, e))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(nets))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors[0]


def test_empty_commit_and_bad_record():
    n = 100
    ty = torch.zeros(n, dtype=torch.uint8, device="cuda")
    z = torch.zeros(n, dtype=torch.int32, device="cuda")
    off = torch.zeros(n + 1, dtype=torch.int64, device="cuda")
    syn = msp.commit_synapses(torch.empty(0, dtype=torch.int32, device="cuda"), off, ty, z,
                              z.clone(), z.clone(), 1, 0, syn_capacity=10)
    assert syn["n_formed"] == 0 and syn["syn_src"].numel() == 0
    net = msp.Network(z, z, z, 8)
    one = lambda *x: torch.tensor(x, dtype=torch.int32, device="cuda")
    net.record(one(0, 1, 2), one(3, 4, 5), torch.zeros(3, dtype=torch.uint8, device="cuda"))
    assert net.m == 3 and net.src[:3].tolist() == [0, 1, 2] and net.tgt[:3].tolist() == [3, 4, 5]
    with pytest.raises(msp.MspError):
        net.record(one(0, n), one(3, 4), torch.zeros(2, dtype=torch.uint8, device="cuda"))
