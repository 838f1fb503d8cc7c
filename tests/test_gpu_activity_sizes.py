"""The activity run at the sizes where it can go wrong: no synapses at all, neurons with one to
many synapses (read four at a time), blocks of neurons and of approximated synapses cut
short, epochs that close in a run's first or last step, with the approximated synapses of a
step taken with the step before or by themselves: bitwise against the oracle."""
import numpy as np
import pytest
import torch

import paper_2509_26193_amd as msp
from gpu_util import T
from test_gpu_activity import _net, _pair, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,m,approx,t0,steps", [
    (1, 0, 0, 0, 3), (1, 3, 0, 0, 5), (33, 1000, 0, 98, 4), (300, 5000, 1, 97, 6),
    (257, 2600, 2, 99, 2), (5000, 20000, 2, 95, 5), (5000, 20000, 1, 99, 1),
    (255, 1048577, 0, 98, 3), (256, 1048577, 1, 98, 3), (256, 1048577, 2, 97, 4),
    (1048577, 0, 0, 99, 2), (1048609, 1500000, 1, 97, 5)])
def test_activity_matches_oracle(n, m, approx, t0, steps):
    ty, src, tgt, sty, rank = _net(n, m, seed=n % 1000 + m % 7)
    if m > 100:                                  # one neuron with many synapses, on few targets
        src[: min(m // 2, 70)] = 0
        tgt[: min(m // 2, 70)] = n - 1
        sty = ty[src].copy()
    g, o = _pair(ty, seed=n % 91, spk_share=0.3, freq_hi=0.3)
    g.spiked[0] = 1
    o.spk[0] = 1
    spikes = torch.zeros(1, dtype=torch.int64, device="cuda")
    li_g = g.run(T(src, torch.int32), T(tgt, torch.int32), T(sty, torch.uint8), seed=3, t0=t0,
                 steps=steps, approx=approx, rank=T(rank, torch.int32), last_input=True,
                 spikes=spikes)
    total, li_o = o.run(src, tgt, sty, seed=3, t0=t0, steps=steps, approx=approx, rank=rank,
                        last_input=True)
    assert int(spikes.item()) == total
    _same(g, o, li_g, li_o, (n, m, approx))
