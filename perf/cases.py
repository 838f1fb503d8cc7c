"""Cases of the framework's performance measurements: what a simulation of structural
plasticity has the library do, from one update of a few thousand neurons to one of
2^23. Sizes, densities and options are those of the repository's workloads
(synth_inputs, bench.py, the tests) and sizes between them, odd ones among them.

A case is a dict of plain values with a "kind":

  update    one whole connectivity update from the positions: octree, vacancy refresh,
            target search, acceptance of the requests, recording of the synapses (the first
            update of a run)
  search    refresh and target search on a kept octree, where only a share of the neurons
            still has vacant axonal elements (a later update of a run), in one phase or
            in the two phases of the location-aware form
  cycle     whole updates of a running network as a plan replays them: refresh, search,
            acceptance, recording, growth, deletion and retraction
  batch     the search of many simulations of an ensemble in one replayed plan
  attract   expected attraction and its gradients in the positions and sigma (one step of
            an optimisation through the differentiated form)
  activity  electrical activity between two updates, every spike exchanged (approx 0) or
            frequencies between ranks (1) or everywhere (2)

Inputs are drawn on the GPU from the seed: positions uniform in a cube or in Gaussian
clusters, four neurons of five excitatory, zero to a few vacant elements per neuron.
exact() evaluates the floating-point outputs in float64 with torch alone.
"""
import math

import torch

import paper_2509_26193_amd as msp

DEV = "cuda"
SIGMA = 750.0


# ----------------------------------------------------------------------------- the cases
def _edge(n, per_4096=1000.0):
    """Edge of a cube that holds n neurons at the density of 4096 in `per_4096` um."""
    return round(per_4096 * (n / 4096.0) ** (1.0 / 3.0), 1)


def listed():
    return [
        # the smallest whole update: the first update of a network of a few thousand
        # neurons, where launches and host waits count
        dict(name="update_4096", kind="update", n=4096, layout="uniform", edge=1000.0, theta=0.3,
             a_hi=2, v_hi=3),
        # an ordinary network of odd size at the finest accuracy that is used
        dict(name="update_60001", kind="update", n=60001, layout="uniform", edge=_edge(60001),
             theta=0.2, a_hi=2, v_hi=3),
        # a clustered network of a million neurons: deep, uneven octree, more requests
        # per target
        dict(name="update_clusters_1048576", kind="update", n=1048576, layout="clusters",
             edge=10000.0, theta=0.3, a_hi=4, v_hi=4),
        # the largest: one GPU's share of a large simulation, as the benchmark runs it
        dict(name="update_8388608", kind="update", n=8388608, layout="uniform", edge=20000.0,
             theta=0.3, a_hi=2, v_hi=3),
        # a later update of a large network: about one neuron in eight still searches
        dict(name="search_sparse_1500007", kind="search", n=1500007, layout="uniform",
             edge=_edge(1500007), theta=0.3, share=0.12, branch_level=0),
        # a small running network: its updates are launches and short kernels
        dict(name="cycle_20011", kind="cycle", n=20011, edge=_edge(20011), theta=0.3, updates=2),
        # a large running network
        dict(name="cycle_2097152", kind="cycle", n=2097152, edge=_edge(2097152), theta=0.3,
             updates=2),
        # an ensemble of small and middling simulations, replayed from a plan that was tuned
        dict(name="batch_64", kind="batch", sims=64, log2_lo=12, log2_hi=18, theta=0.3, tuned=True),
        # gradients of a small network, and of the largest the repository differentiates
        dict(name="attract_10007", kind="attract", n=10007, edge=_edge(10007), theta=0.3),
        dict(name="attract_262144", kind="attract", n=262144, edge=5000.0, theta=0.3),
        # the epoch of 100 steps between two updates: a middling network whose ranks
        # exchange frequencies, and part of one of the largest with every spike exchanged
        dict(name="activity_131101", kind="activity", n=131101, per_neuron=2.0, steps=100,
             approx=1),
        dict(name="activity_8388608", kind="activity", n=8388608, per_neuron=0.9, steps=20,
             approx=0),
    ]


def _size(rng, lo, hi):
    """A size spread over the logarithm of [lo, hi], half of them odd."""
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return min(hi, n | 1) if rng.random() < 0.5 else n


def draw(rng):
    kind = rng.choice(["update", "update", "search", "cycle", "batch", "attract", "activity"])
    theta = rng.choice([0.2, 0.25, 0.3, 0.3, 0.4, 0.5])
    if kind == "update":
        clusters = rng.random() < 0.35
        if clusters:
            n = _size(rng, 8192, 1 << 20)
            return dict(kind=kind, n=n, layout="clusters", edge=_edge(n, 1575.0), theta=theta,
                        a_hi=4, v_hi=4)
        n = _size(rng, 1500, 3 << 20)
        return dict(kind=kind, n=n, layout="uniform", edge=_edge(n, rng.choice([1000.0, 1575.0])),
                    theta=theta, a_hi=rng.choice([1, 2, 2, 3]), v_hi=rng.choice([1, 3, 3, 5]))
    if kind == "search":
        n = _size(rng, 4000, 2 << 20)
        return dict(kind=kind, n=n, layout=rng.choice(["uniform", "uniform", "clusters"]),
                    edge=_edge(n), theta=theta, share=round(rng.uniform(0.02, 0.6), 3),
                    branch_level=rng.choice([0, 0, 3, 5]))
    if kind == "cycle":
        n = _size(rng, 2000, 2 << 20)
        return dict(kind=kind, n=n, edge=_edge(n), theta=max(theta, 0.25),
                    updates=rng.choice([1, 2, 3]))
    if kind == "batch":
        lo = rng.choice([10, 12, 12])
        return dict(kind=kind, sims=rng.choice([3, 8, 17, 32, 50]), log2_lo=lo,
                    log2_hi=rng.choice([14, 16, 17]), theta=max(theta, 0.25),
                    tuned=rng.random() < 0.5)
    if kind == "attract":
        n = _size(rng, 1500, 200000)
        return dict(kind=kind, n=n, edge=_edge(n, rng.choice([1000.0, 1250.0])),
                    theta=max(theta, 0.25))
    n = _size(rng, 5000, 4 << 20)
    return dict(kind=kind, n=n, per_neuron=round(rng.uniform(0.5, 4.0), 2),
                steps=rng.choice([10, 25, 50]), approx=rng.choice([0, 0, 1, 2]))


# ----------------------------------------------------------------------------- inputs
class _Gen:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(int(seed))

    def uniform(self, *shape):
        return torch.rand(shape, generator=self.g, dtype=torch.float64, device=DEV)

    def normal(self, *shape):
        return torch.randn(shape, generator=self.g, dtype=torch.float64, device=DEV)

    def ints(self, n, hi, dtype=torch.int32):
        """n integers of 0..hi."""
        return torch.randint(0, hi + 1, (n,), generator=self.g, device=DEV).to(dtype)

    def types(self, n):
        """Four of five neurons excitatory (0), at random places."""
        t = torch.ones(n, dtype=torch.uint8, device=DEV)
        p = torch.randperm(n, generator=self.g, device=DEV)
        t[p[: int(round(0.8 * n))]] = 0
        return t


def _positions(g, n, layout, edge):
    """(pos [n][3], box_min, box_edge)."""
    if layout == "uniform":
        return g.uniform(n, 3) * edge, [0.0, 0.0, 0.0], float(edge)
    centres = g.uniform(64, 3) * edge
    at = torch.arange(n, device=DEV) % 64
    pos = centres[at] + g.normal(n, 3) * (0.015 * edge)
    lo = pos.min(dim=0).values
    L = float((pos.max(dim=0).values - lo).max().item())
    return pos, [float(x) for x in lo.tolist()], L


def _counts(g, n, a_hi, v_hi):
    return g.ints(n, a_hi), g.ints(n, v_hi), g.ints(n, v_hi)


def _room(mean):
    """Room for a number of elements whose mean over the inputs is `mean`."""
    return int(1.1 * mean) + 256


def _network(va, ve, vi, room):
    """A network without synapses, with room for `room` of them."""
    net = msp.Network(va, ve, vi, room)
    for x in (net.src, net.tgt, net.type):
        x.zero_()
    return net


def _batch_sizes(case):
    """The simulations' sizes: spread over the logarithm of the range (golden-ratio steps)."""
    lo, hi = case["log2_lo"], case["log2_hi"]
    return [int(round(2.0 ** (lo + (hi - lo) * ((0.5 + k * 0.6180339887498949) % 1.0))))
            for k in range(case["sims"])]


def prepare(case, seed):
    return globals()["_prepare_" + case["kind"]](case, seed)


def run(state):
    return globals()["_run_" + state["kind"]](state)


def _prepare_update(case, seed):
    g, n = _Gen(seed), case["n"]
    pos, box_min, box_edge = _positions(g, n, case["layout"], case["edge"])
    ty = g.types(n)
    va0, ve0, vi0 = _counts(g, n, case["a_hi"], case["v_hi"])
    room = _room(n * case["a_hi"] / 2.0)
    return dict(kind="update", pos=pos, box_min=box_min, box_edge=box_edge, ty=ty, va0=va0,
                ve0=ve0, vi0=vi0, va=va0.clone(), ve=ve0.clone(), vi=vi0.clone(), room=room,
                net=_network(va0, ve0, vi0, room),
                target=torch.full((room,), -1, dtype=torch.int32, device=DEV),
                offset=torch.empty(n + 1, dtype=torch.int64, device=DEV),
                theta=case["theta"], seed=seed)


def _run_update(st):
    tree = msp.build_octree(st["pos"], st["box_min"], st["box_edge"])
    va, ve, vi, net = st["va"], st["ve"], st["vi"], st["net"]
    net.m = 0                               # a network without synapses
    net.bound.zero_()
    va.copy_(st["va0"])
    ve.copy_(st["ve0"])
    vi.copy_(st["vi0"])
    msp.update_vacant_counts(tree, ve, vi)
    tgt, off = msp.find_targets(tree, st["ty"], va, SIGMA, st["theta"], st["seed"], 0,
                                target_out=st["target"], elem_offset_out=st["offset"])
    syn = msp.commit_synapses(tgt, off, st["ty"], va, ve, vi, st["seed"], 0,
                              syn_capacity=st["room"])
    net.record(syn["syn_src"], syn["syn_tgt"], syn["syn_type"])
    tree.free()
    return dict(target=st["target"], offset=off, syn_src=net.src, syn_tgt=net.tgt,
                syn_type=net.type, bound=net.bound, vac_axon=va, vac_exc=ve, vac_inh=vi)


def _prepare_search(case, seed):
    g, n = _Gen(seed), case["n"]
    pos, box_min, box_edge = _positions(g, n, case["layout"], case["edge"])
    ty = g.types(n)
    a, ve, vi = _counts(g, n, 1, 3)
    va = (a + 1) * (g.uniform(n) < case["share"]).to(torch.int32)
    tree = msp.build_octree(pos, box_min, box_edge)
    return dict(kind="search", tree=tree, ty=ty, va=va, ve=ve, vi=vi, theta=case["theta"],
                seed=seed, step=0, branch=case["branch_level"],
                target=torch.full((_room(1.5 * n * case["share"]),), -1, dtype=torch.int32,
                                  device=DEV),
                offset=torch.empty(n + 1, dtype=torch.int64, device=DEV))


def _run_search(st):
    msp.update_vacant_counts(st["tree"], st["ve"], st["vi"])
    tgt, off = msp.find_targets(st["tree"], st["ty"], st["va"], SIGMA, st["theta"], st["seed"],
                                st["step"], target_out=st["target"],
                                elem_offset_out=st["offset"], branch_level=st["branch"])
    st["step"] += 1
    return dict(target=st["target"], offset=off)


CYCLE_WARM = 6                  # updates a network has behind it when it is measured


def _prepare_cycle(case, seed):
    g, n = _Gen(seed), case["n"]
    pos, box_min, box_edge = _positions(g, n, "uniform", case["edge"])
    ty = g.types(n)
    va, ve, vi = _counts(g, n, 2, 3)
    tree = msp.build_octree(pos, box_min, box_edge)
    net = _network(va, ve, vi, 4 * n)
    cyc = msp.Cycle(tree, ty, net, va, ve, vi, SIGMA, case["theta"], seed, graph=True)
    cyc.run(CYCLE_WARM)
    assert cyc.status() == 0
    return dict(kind="cycle", cyc=cyc, net=net, tree=tree, updates=case["updates"],
                seen=[torch.empty_like(x) for x in (net.src, net.tgt, net.type)])


def _run_cycle(st):
    st["cyc"].run(st["updates"])
    st["cyc"].counts()          # once per pass, the host learns the length of the list
    net = st["net"]
    for kept, x in zip(st["seen"], net.synapses()):     # the list as it now is, for the record
        kept.zero_()
        kept[:x.numel()].copy_(x)
    src, tgt, sty = st["seen"]
    va, ve, vi = st["cyc"].va_ve_vi()
    return dict(z=net.z, bound=net.bound, src=src, tgt=tgt, type=sty, va=va, ve=ve, vi=vi)


def _prepare_batch(case, seed):
    g = _Gen(seed)
    sims, keep, where = [], [], 0
    for k, n in enumerate(_batch_sizes(case)):
        pos, box_min, box_edge = _positions(g, n, "uniform", _edge(n))
        ty = g.types(n)
        va, ve, vi = _counts(g, n, 2, 3)
        tree = msp.build_octree(pos, box_min, box_edge)
        msp.update_vacant_counts(tree, ve, vi)
        S = _room(n)
        sims.append(dict(tree=tree, neuron_type=ty, vac_axon=va,
                         sigma=500.0 + 500.0 * ((k * 0.7548776662466927) % 1.0), seed=seed + k))
        keep.append((where, S))
        where += (S + 63) // 64 * 64
    out = torch.full((max(where, 1),), -1, dtype=torch.int32, device=DEV)
    for d, (at, S) in zip(sims, keep):      # one buffer for the whole ensemble's targets
        d["target_out"] = out[at:at + S]
    b = msp.Batch(sims, graph=True, autotune=case["tuned"])
    b.run(case["theta"], 0)                 # tunes the plan and captures it
    return dict(kind="batch", b=b, out=out, theta=case["theta"], step=1)


def _run_batch(st):
    st["b"].run(st["theta"], st["step"])
    st["step"] += 1
    return dict(target=st["out"])


def _attract_inputs(case, seed):
    g, n = _Gen(seed), case["n"]
    pos, box_min, box_edge = _positions(g, n, "uniform", case["edge"])
    ty = g.types(n)
    va, ve, vi = _counts(g, n, 2, 3)
    gZ = ((0.5 + g.uniform(n)) * (va > 0)).to(torch.float32)    # dLoss/dZ from further on
    return pos, box_min, box_edge, ty, va, ve, vi, gZ


def _prepare_attract(case, seed):
    pos, box_min, box_edge, ty, va, ve, vi, gZ = _attract_inputs(case, seed)
    tree = msp.build_octree(pos, box_min, box_edge)
    msp.update_vacant_counts(tree, ve, vi)
    sigma = torch.tensor(SIGMA, dtype=torch.float64, device=DEV, requires_grad=True)
    return dict(kind="attract", pos=pos.requires_grad_(True), sigma=sigma, tree=tree, ty=ty, va=va,
                gZ=gZ, theta=case["theta"])


def _run_attract(st):
    Z = msp.attraction(st["pos"], st["sigma"], st["tree"], st["ty"], st["va"], st["theta"])
    dpos, dsigma = torch.autograd.grad(Z, (st["pos"], st["sigma"]), st["gZ"])
    return dict(Z=Z.detach(), dpos=dpos, dsigma=dsigma)


def _activity_inputs(case, seed):
    """Types, ranks, synapses and the running state of the neurons (about 15 Hz)."""
    g, n = _Gen(seed), case["n"]
    ty = g.types(n)
    rank = (torch.arange(n, device=DEV) * 8 // n).to(torch.int32)
    m = int(n * case["per_neuron"])
    src, tgt = g.ints(m, n - 1), g.ints(m, n - 1)
    near = g.uniform(m) < 0.9               # most partners lie in the same rank
    tgt = torch.where(near, ((src + tgt % 512).clamp(max=n - 1)).to(torch.int32), tgt)
    sty = ty[src.long()].contiguous()
    v = -75.0 + 25.0 * g.uniform(n)
    u = torch.where(ty == 0, -13.0 + 6.0 * g.uniform(n), -14.0 + 3.0 * g.uniform(n))
    calcium = 0.1 + 0.1 * g.uniform(n)
    spiked = (g.uniform(n) < 0.015).to(torch.uint8)
    count = g.ints(n, 2)
    freq = g.ints(n, 4).to(torch.float64) * 0.01
    return ty, rank, src, tgt, sty, dict(v=v, u=u, calcium=calcium, spiked=spiked, count=count,
                                         freq=freq)


def _prepare_activity(case, seed):
    ty, rank, src, tgt, sty, s = _activity_inputs(case, seed)
    act = msp.Activity(ty)
    for k, x in s.items():
        getattr(act, k).copy_(x)
    return dict(kind="activity", act=act, rank=rank, src=src, tgt=tgt, sty=sty, seed=seed,
                approx=case["approx"], steps=case["steps"], t=0,
                spikes=torch.zeros(1, dtype=torch.int64, device=DEV))


def _run_activity(st):
    act = st["act"]
    act.run(st["src"], st["tgt"], st["sty"], st["seed"], st["t"], st["steps"],
            approx=st["approx"], rank=st["rank"], spikes=st["spikes"])
    st["t"] += st["steps"]
    return dict(v=act.v, u=act.u, calcium=act.calcium, spiked=act.spiked, count=act.count,
                freq=act.freq, spikes=st["spikes"])


# ----------------------------------------------------------------------------- work
def _search_work(sources, searches, n, theta):
    """Bytes and operations of `searches` searches from `sources` neurons among n: the
    level-0 list of a source has about 360 records per doubling of n at theta = 0.3, and
    grows as theta^-2.6; 11 operations each. Per source its position and type, per
    search its target."""
    visits = min(1.3 * n, max(50.0, 360.0 * (math.log2(n) - 9.2)) * (0.3 / theta) ** 2.6)
    return 29.0 * sources + 4.0 * searches, 11.0 * visits * sources


def work(case):
    kind = case["kind"]
    if kind == "batch":
        b = f = 0.0
        for n in _batch_sizes(case):
            x, y = _search_work(n * 2 / 3, n, n, case["theta"])
            b, f = b + x + 12.0 * n + 1.3 * n * 64, f + y
        return dict(bytes=b, flops=f)
    n = case["n"]
    nodes = 1.3 * n
    refresh = 8.0 * n + 24.0 * n + 2 * 32.0 * nodes      # counts and positions in, records out
    if kind == "update":
        S = n * case["a_hi"] / 2.0
        x, y = _search_work(n * case["a_hi"] / (case["a_hi"] + 1.0), S, n, case["theta"])
        # positions in, keys and order out; vacancies in and out; offsets; synapses
        return dict(bytes=36.0 * n + refresh + x + 33.0 * n + 4.0 * S + 9.0 * S, flops=y)
    if kind == "search":
        src = n * case["share"]
        x, y = _search_work(src, 1.5 * src, n, case["theta"])
        return dict(bytes=refresh + x + 12.0 * n, flops=y)
    if kind == "cycle":
        x, y = _search_work(0.12 * n, 0.14 * n, n, case["theta"])
        # element counts and bound elements in and out, vacancies out, the list read and
        # written once
        per = refresh + x + 2 * 36.0 * n + 12.0 * n + 2 * 9.0 * n
        return dict(bytes=per * case["updates"], flops=y * case["updates"])
    if kind == "attract":
        x, y = _search_work(n * 2 / 3, 0, n, case["theta"])
        # forward, backward: the sums once more with 7 operations per accepted record
        return dict(bytes=2 * (x + nodes * 64) + 4.0 * n + 12.0 * n + 4.0 * n, flops=2.6 * y)
    m = n * case["per_neuron"]
    per = 57.0 * n + 0.015 * 13.0 * m + (17.0 * m if case["approx"] == 2 else
                                         1.7 * m if case["approx"] == 1 else 0.0)
    # per step and neuron: the Philox draw (about 200 operations) and the model (30)
    return dict(bytes=per * case["steps"], flops=230.0 * n * case["steps"])


# ----------------------------------------------------------------------------- exact
M32 = 0xFFFFFFFF


def _mulhilo(a, b):
    """High and low 64 bits of a * b (a: a Python integer; int64 tensors hold the bits)."""
    al, ah = a & M32, a >> 32
    bl, bh = b & M32, (b >> 32) & M32
    ll, lh, hl, hh = bl * al, bh * al, bl * ah, bh * ah
    mid = ((ll >> 32) & M32) + (lh & M32) + (hl & M32)
    hi = hh + ((lh >> 32) & M32) + ((hl >> 32) & M32) + ((mid >> 32) & M32)
    lo = (ll & M32) | (mid << 32)
    return hi, lo


def _signed(x):
    x &= (1 << 64) - 1
    return x - (1 << 64) if x >> 63 else x


def _philox(c0, c1, c2, c3, k0, k1, dev):
    """Philox4x64-10 words 0 and 1 (Salmon et al., SC'11) as int64 tensors."""
    t = [torch.as_tensor(_signed(c) if isinstance(c, int) else c, dtype=torch.int64, device=dev)
         for c in (c0, c1, c2, c3)]
    k0, k1 = int(k0), int(k1)
    for _ in range(10):
        h0, l0 = _mulhilo(0xD2E7470EE14C6C93, t[0])
        h1, l1 = _mulhilo(0xCA5A826395121157, t[2])
        t = [h1 ^ t[1] ^ _signed(k0), l1, h0 ^ t[3] ^ _signed(k1), l0]
        k0 = (k0 + 0x9E3779B97F4A7C15) & ((1 << 64) - 1)
        k1 = (k1 + 0xBB67AE8584CAA73B) & ((1 << 64) - 1)
    return t[0], t[1]


def _unit53(w):
    """(w >> 11) 2^-53 of unsigned 64-bit words."""
    return ((w >> 11) & ((1 << 53) - 1)).to(torch.float64) * 2.0 ** -53


def exact(case, seed):
    f = globals().get("_exact_" + case["kind"])
    return f(case, seed) if f else None         # the other kinds return whole numbers only


def _exact_cycle(case, seed):
    """The element counts after the warm-up and one pass (the growth rule; they do not
    depend on the synapses)."""
    g, n = _Gen(seed), case["n"]
    _positions(g, n, "uniform", case["edge"])
    g.types(n)
    z = torch.stack(_counts(g, n, 2, 3)).to(torch.float64)
    p = msp.PLASTICITY
    xi = 0.5 * (p["growth_onset"] + p["target_calcium"])
    zeta = (p["target_calcium"] - p["growth_onset"]) / (2.0 * math.sqrt(math.log(2.0)))
    j = torch.arange(n, dtype=torch.int64, device=DEV)
    for step in range(CYCLE_WARM + case["updates"]):
        for k in range(3):
            w0, w1 = _philox(j, k, step, 0, seed, 2, DEV)
            u1 = (((w0 >> 11) & ((1 << 53) - 1)) + 1).to(torch.float64) * 2.0 ** -53
            gauss = torch.sqrt(-2.0 * torch.log(u1)) * torch.cos(2.0 * math.pi * _unit53(w1))
            r = (p["calcium_mean"] + p["calcium_sd"] * gauss - xi) / zeta
            dz = p["steps_per_update"] * p["growth_rate"] * (2.0 * torch.exp(-r * r) - 1.0)
            z[k] = (z[k] + dz).clamp(min=0.0)
    return dict(z=z)


def _exact_activity(case, seed):
    ty, rank, src, tgt, sty, s = _activity_inputs(case, seed)
    P, n = msp.ACTIVITY, case["n"]
    exc = ty == 0
    par = {k: torch.where(exc, torch.tensor(P[k + "_exc"], dtype=torch.float64, device=DEV),
                          torch.tensor(P[k + "_inh"], dtype=torch.float64, device=DEV))
           for k in "abcd"}
    inv_tau, inv_delta = 1.0 / P["ca_tau"], 1.0 / P["epoch"]
    src, tgt = src.long(), tgt.long()
    if case["approx"] == 1:
        remote = rank[src] != rank[tgt]
    else:
        remote = torch.full_like(src, case["approx"] == 2, dtype=torch.bool)
    at = torch.nonzero(remote).squeeze(1)
    gid = torch.arange(n, dtype=torch.int64, device=DEV)
    v, u, ca, spk, cnt, freq = (s[k].clone() for k in ("v", "u", "calcium", "spiked", "count",
                                                       "freq"))
    total = 0
    for t in range(case["steps"]):
        fire = (spk[src] != 0) & ~remote
        if at.numel():
            fire[at] = _unit53(_philox(at, t, 0, 0, seed, 5, DEV)[0]) < freq[src[at]]
        q = torch.nonzero(fire).squeeze(1)
        e = torch.bincount(tgt[q][sty[q] == 0], minlength=n).to(torch.float64)
        h = torch.bincount(tgt[q][sty[q] == 1], minlength=n).to(torch.float64)
        uu = _unit53(_philox(gid, t, 0, 0, seed, 6, DEV)[0])
        I = P["w_exc"] * e - P["w_inh"] * h + (P["bg_mean"] + P["bg_width"] * (uu - 0.5))
        for _ in range(2):
            v = v + 0.5 * (0.04 * v * v + 5.0 * v + 140.0 - u + I)
        u = u + par["a"] * (par["b"] * v - u)
        f = v >= 30.0
        v = torch.where(f, par["c"], v)
        u = torch.where(f, u + par["d"], u)
        ca = ca - ca * inv_tau
        ca = torch.where(f, ca + P["ca_beta"], ca)
        spk = f.to(torch.uint8)
        cnt = cnt + f.to(torch.int32)
        if (t + 1) % P["epoch"] == 0:
            freq = cnt.to(torch.float64) * inv_delta
            cnt = torch.zeros_like(cnt)
        total += int(f.sum().item())
    return dict(v=v, u=u, calcium=ca, freq=freq)


def _spread(q):
    """Every third bit of a 21-bit number."""
    out = torch.zeros_like(q)
    for b in range(21):
        out |= ((q >> b) & 1) << (3 * b)
    return out


def _exact_attract(case, seed):
    """Z, dpos and dsigma by a breadth-first Barnes-Hut expansion in float64."""
    pos, box_min, L, ty, va, ve, vi, gZ = _attract_inputs(case, seed)
    n, theta, s2 = case["n"], case["theta"], SIGMA * SIGMA
    q = torch.floor((pos - torch.tensor(box_min, dtype=torch.float64, device=DEV)) / L * 2097152.0)
    q = q.clamp(0, 2097151).to(torch.int64)
    key = (_spread(q[:, 0]) << 2) | (_spread(q[:, 1]) << 1) | _spread(q[:, 2])
    key, order = torch.sort(key, stable=True)
    sp = pos[order]
    begin, cell_of = [], []                 # per depth: the cells' first places; each place's cell
    for k in range(22):
        p = key >> (3 * (21 - k))
        new = torch.ones(n, dtype=torch.bool, device=DEV)
        new[1:] = p[1:] != p[:-1]
        begin.append(torch.nonzero(new).squeeze(1))
        cell_of.append(torch.cumsum(new.to(torch.int64), 0) - 1)
        if begin[-1].numel() == n:
            break
    depths = len(begin)
    Z = torch.zeros(n, dtype=torch.float64, device=DEV)
    dpos = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
    dsigma = torch.zeros((), dtype=torch.float64, device=DEV)
    place = torch.empty(n, dtype=torch.int64, device=DEV)
    place[order] = torch.arange(n, device=DEV)
    for t in (0, 1):
        w = (vi if t else ve)[order].to(torch.float64)
        vs, cs, Gs = [], [], []
        for k in range(depths):
            C = begin[k].numel()
            v = torch.zeros(C, dtype=torch.float64, device=DEV).index_add_(0, cell_of[k], w)
            c = torch.zeros(C, 3, dtype=torch.float64, device=DEV)
            c.index_add_(0, cell_of[k], sp * w[:, None])
            vs.append(v)
            cs.append(c / v.clamp(min=1.0)[:, None])
            Gs.append(torch.zeros(C, 3, dtype=torch.float64, device=DEV))
        sources = torch.nonzero((va > 0) & (ty == t)).squeeze(1)
        for i0 in range(0, sources.numel(), 16384):
            src = sources[i0:i0 + 16384]
            cell = torch.zeros_like(src)    # every source opens the root
            for k in range(1, depths):
                if not src.numel():
                    break
                first = begin[k - 1][cell]
                last = torch.full_like(first, n)
                inner = cell + 1 < begin[k - 1].numel()
                last[inner] = begin[k - 1][cell[inner] + 1]
                c0 = cell_of[k][first]
                many = cell_of[k][last - 1] - c0 + 1
                src = torch.repeat_interleave(src, many)
                ends = torch.cumsum(many, 0)
                cell = torch.repeat_interleave(c0 - (ends - many), many) + torch.arange(
                    src.numel(), device=DEV)
                keep = vs[k][cell] > 0
                src, cell = src[keep], cell[keep]
                first = begin[k][cell]
                last = torch.full_like(first, n)
                inner = cell + 1 < begin[k].numel()
                last[inner] = begin[k][cell[inner] + 1]
                leaf = last - first == 1
                home = (place[src] >= first) & (place[src] < last)
                d = pos[src] - cs[k][cell]
                d2 = d.square().sum(dim=1)
                l = L * 2.0 ** -k
                take = torch.where(leaf, ~home, ~home & (l * l < theta * theta * d2))
                a, b, da, d2a = src[take], cell[take], d[take], d2[take]
                wt = vs[k][b] * torch.exp(-d2a / s2)
                Z.index_add_(0, a, wt)
                gw = gZ[a].to(torch.float64) * wt
                fd = (gw * (2.0 / s2))[:, None] * da
                Gs[k].index_add_(0, b, fd)
                dpos.index_add_(0, a, -fd)
                dsigma = dsigma + (gw * d2a).sum() * (2.0 / (s2 * SIGMA))
                go = ~take & ~leaf
                src, cell = src[go], cell[go]
        H = torch.zeros(n, 3, dtype=torch.float64, device=DEV)
        for k in range(1, depths):
            part = Gs[k] / vs[k].clamp(min=1.0)[:, None]
            alone = torch.diff(begin[k - 1], append=torch.tensor([n], device=DEV)) == 1
            H += torch.where(alone[cell_of[k - 1]][:, None], torch.zeros_like(H), part[cell_of[k]])
        dpos.index_add_(0, order, H * w[:, None])
    return dict(Z=Z, dpos=dpos, dsigma=dsigma)
