"""Timed cases: the work that programs built on this library have it do, through its public
entry points, from one small instance to the largest batch and lattice.

A sampler case is a batch of instances whose context has finished tuning and burn-in; a pass
runs a block of parallel-tempering cycles and reads the results a program would act on: every
instance's observables, and where the configurations themselves are wanted the spins.  A
network case is one training step or one forward pass of the ladder network.

Couplings, fields, spins and parameters come from the seed.  The graphs (and their colourings)
come from the case alone, as disorder realisations of one lattice or graph ensemble do.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import workloads as W
from paper_1004_0023_amd import ptqmc

GRAPH_SEED = 20100401
# Cycles before the timed passes: longer than the launch-shape tuning of either encoding, and
# the burn-in every program discards.  A fixed number, so that a state depends on the case
# and the seed only.
BURN_IN = 48
KEYS = ("E_cl", "C", "rung_of", "replica_of", "acc", "att", "roundtrips", "label", "sumE", "sumC",
        "sumE2", "sumC2", "nup", "ndown")


def _sampler(name=None, *, graph="regular", n=0, n_max=0, degree=0, degree_max=0, m=0, r=0, jmax=1,
             hmax=1, gamma=1.0, t_min=0.1, t_max=3.0, instances=1, graphs=1, k=10, cycles=1,
             encoding="int8", tau=False, spins=False):
    case = {"kind": "sampler", "graph": graph, "n": n, "n_max": n_max or n, "degree": degree,
            "degree_max": degree_max or degree, "m": m, "r": r, "jmax": jmax, "hmax": hmax,
            "gamma": gamma, "t_min": t_min, "t_max": t_max, "instances": instances,
            "graphs": min(graphs, instances), "k": k, "cycles": cycles, "encoding": encoding,
            "tau": tau, "spins": spins}
    return case if name is None else dict(case, name=name)


def _network(name=None, *, op, batch, loss="sigmoid"):
    case = {"kind": "network", "op": op, "batch": batch, "loss": loss}
    return case if name is None else dict(case, name=name)


def listed():
    return [
        # One 8-spin instance, an exchange after every sweep: interactive use, where a pass is
        # launch and read-back latency.
        _sampler("tiny_bytes", n=8, degree=3, m=16, r=8, t_max=2.0, k=1, cycles=16),
        # One weighted 128-spin problem on 32 rungs: a single instance that cannot fill the chip.
        _sampler("single_bytes", n=128, degree=6, m=64, r=32, jmax=3, hmax=0, t_min=0.05, cycles=16),
        # The batched workload: 512 uneven instances in one context, 32 replicas to a word,
        # read out between long blocks of cycles.
        _sampler("batch_packed", graph="ensemble", instances=512, graphs=128, cycles=50,
                 encoding="bitpack"),
        # The same ensemble one byte per spin (the default encoding), a quarter of the batch.
        _sampler("batch_bytes", graph="ensemble", instances=128, graphs=128, cycles=50),
        # A 1024-site periodic cubic lattice with 256 slices, and its configurations.
        _sampler("lattice_packed", graph="cubic", n=8 * 8 * 16, m=256, r=64, hmax=0, gamma=1.5,
                 t_min=0.2, t_max=2.0, cycles=64, encoding="bitpack", spins=True),
        # The same lattice in bytes with imaginary-time correlations at every exchange (gaps).
        _sampler("lattice_correlations", graph="cubic", n=8 * 8 * 16, m=256, r=64, hmax=0, gamma=1.5,
                 t_min=0.2, t_max=2.0, cycles=32, tau=True),
        # A classical +-1 spin glass (M = 1): 16 disorder realisations of a 10^3 lattice and
        # the configurations found.
        _sampler("classical_bytes", graph="cubic", n=1000, m=1, r=32, hmax=0, t_min=0.2, t_max=2.0,
                 instances=16, cycles=64, spins=True),
        # A slice count chosen for its Trotter error rather than as a power of two, an odd
        # number of sites, an odd ladder.
        _sampler("slices_bytes", n=201, degree=4, m=100, r=27, jmax=2, hmax=2, instances=8, graphs=8,
                 cycles=16),
        # Weighted couplings and fields in the packed encoding.
        _sampler("weighted_packed", n=128, degree=6, m=64, r=48, jmax=3, hmax=3, instances=16, graphs=16,
                 cycles=32, encoding="bitpack"),
        # Open boundaries (sites of three to six neighbours), packed, with configurations.
        _sampler("open_packed", graph="open", n=6 * 7 * 8, m=64, r=40, gamma=1.2, t_min=0.2,
                 instances=8, cycles=32, encoding="bitpack", spins=True),
        # One step of training the ladder network at its batch size: loss, gradients, Adam.
        _network("network_training", op="train", batch=256),
        # Ladders for a whole batch of instances.
        _network("network_inference", op="forward", batch=512),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["small", "batch", "lattice", "classical", "slices", "packed", "network"],
                       weights=[2, 2, 2, 2, 2, 3, 2])[0]
    if kind == "network":
        return _network(op=rng.choice(["train", "forward"]), batch=_log(rng, 1, 4096),
                        loss=rng.choice(["sigmoid", "softmax"]))
    enc = rng.choice(["int8", "bitpack"])
    if kind == "small":
        n, d = _log(rng, 8, 256), rng.randint(3, 7)
        case = _sampler(n=n + (n * d) % 2, degree=d, m=rng.choice([8, 16, 32, 64, 128]), r=_log(rng, 2, 96),
                        jmax=rng.randint(1, 3), hmax=rng.randint(0, 2), k=rng.randint(1, 10),
                        cycles=_log(rng, 1, 64), encoding="int8")
    elif kind == "batch":
        b = _log(rng, 4, 256)
        case = _sampler(graph="ensemble", instances=b, graphs=min(b, 64), cycles=_log(rng, 2, 32),
                        k=rng.choice([1, 5, 10]), encoding=enc, tau=enc == "int8" and rng.random() < 0.3)
    elif kind == "lattice":
        n = rng.randint(4, 8) * rng.randint(4, 9) * rng.randint(4, 16)
        case = _sampler(graph="cubic", n=n, m=rng.choice([32, 64, 128, 256]), r=_log(rng, 8, 64), hmax=0,
                        gamma=1.5, t_min=0.2, t_max=2.0, cycles=_log(rng, 4, 48), encoding=enc,
                        tau=enc == "int8" and rng.random() < 0.3, spins=rng.random() < 0.5)
    elif kind == "classical":
        n = rng.randint(3, 12) * rng.randint(4, 12) * rng.randint(4, 12)
        case = _sampler(graph=rng.choice(["cubic", "open"]), n=n, m=1, r=_log(rng, 4, 64), jmax=rng.choice([1, 1, 3]),
                        hmax=rng.randint(0, 1), t_min=0.2, t_max=2.0, instances=_log(rng, 1, 32),
                        cycles=_log(rng, 8, 64), encoding=enc, spins=rng.random() < 0.5)
    elif kind == "slices":
        n, d = _log(rng, 16, 300), rng.randint(3, 6)
        case = _sampler(n=n + (n * d) % 2, degree=d, m=2 * rng.randint(3, 80), r=_log(rng, 4, 48),
                        jmax=rng.randint(1, 9), hmax=rng.randint(0, 4), instances=_log(rng, 1, 16), graphs=16,
                        cycles=_log(rng, 4, 16), encoding="int8")
    else:
        n, d = _log(rng, 24, 400), rng.randint(3, 8)
        case = _sampler(graph=rng.choice(["regular", "sparse"]), n=n + (n * d) % 2, degree=d,
                        m=rng.choice([16, 32, 64, 128, 2 * rng.randint(5, 60)]), r=_log(rng, 8, 80),
                        jmax=rng.choice([1, 1, 2, 3]), hmax=rng.randint(0, 3), instances=_log(rng, 1, 16),
                        graphs=16, cycles=_log(rng, 4, 32), encoding="bitpack")
    # no drawn case takes more attempts than these, whatever its family
    most = 1.5e10 if kind in ("batch", "lattice") else 4e8
    per_cycle = _attempts(dict(case, cycles=1))
    case["cycles"] = max(1, min(case["cycles"], int(most / per_cycle)))
    return case


# ------------------------------------------------------------------ inputs

def _sides(n):
    """Three sides of at least three with product n, as equal as may be."""
    best = None
    for a in range(3, int(round(n ** (1 / 3))) + 1):
        if n % a:
            continue
        for b in range(a, int(math.isqrt(n // a)) + 1):
            if (n // a) % b == 0:
                best = (a, b, n // a // b)
    return best if best is not None else (3, 3, n // 9)


@functools.lru_cache(maxsize=512)
def _graph(graph, n, degree, index):
    """(edges, colours) of a graph, labels contiguous in colour."""
    rng = np.random.default_rng([GRAPH_SEED, n, degree, index])
    if graph == "regular":
        edges = W.random_regular_graph(n, degree, rng)
    elif graph == "sparse":  # random pairs, degree at most twice the mean and at most eight
        edges, deg, cap = set(), [0] * n, min(8, 2 * degree)
        while 2 * len(edges) < min(degree, cap - 1) * n * 0.8:
            a, b = sorted(int(v) for v in rng.integers(0, n, 2))
            if a != b and deg[a] < cap and deg[b] < cap and (a, b) not in edges:
                edges.add((a, b))
                deg[a] += 1
                deg[b] += 1
        edges = np.array(sorted(edges), dtype=np.int32)
    else:
        lx, ly, lz = _sides(n)
        n = lx * ly * lz
        edges = W.cubic_lattice(lx, ly, lz)
        if graph == "open":
            xyz = np.stack([edges % lx, edges // lx % ly, edges // (lx * ly)])
            edges = edges[np.abs(xyz[:, :, 0] - xyz[:, :, 1]).sum(0) == 1]
    one = W.make_instance(n, edges, np.ones(len(edges), np.int8), np.zeros(n, np.int8), 2, [1.0, 2.0], 1.0)
    return one.N, one.edges, one.color, one.n_colors


@functools.lru_cache(maxsize=512)
def _ensemble_member(index):
    """Sizes of member `index` of the uneven ensemble: N, degree, M, R."""
    rng = np.random.default_rng([GRAPH_SEED, 3, index])
    n, d = int(rng.integers(32, 513)), int(rng.integers(4, 9))
    return n + (n * d) % 2, d, int(rng.choice([32, 64, 128])), int(rng.choice([16, 32, 64]))


def _shapes(case):
    """(graph kind, N, degree, graph index, M, R) of every instance."""
    out = []
    for i in range(case["instances"]):
        g = i % case["graphs"]
        if case["graph"] == "ensemble":
            n, d, m, r = _ensemble_member(g)
            out.append(("regular", n, d, g, m, r))
        else:
            n = case["n"]
            if case["graph"] in ("cubic", "open"):
                n = math.prod(_sides(n))
            out.append((case["graph"], n, case["degree"], g, case["m"], case["r"]))
    return out


def _instances(case, seed):
    rng = np.random.default_rng([GRAPH_SEED, int(seed)])
    weights = np.array([v for v in range(-case["jmax"], case["jmax"] + 1) if v], dtype=np.int8)
    out = []
    for graph, n, d, g, m, r in _shapes(case):
        n, edges, color, n_colors = _graph(graph, n, d, g)
        T = W.geometric_temperatures(case["t_min"], case["t_max"], r)
        b, K = W.st_rungs(T, case["gamma"], m)
        out.append(W.Instance(N=n, M=m, R=r, edges=edges, J=rng.choice(weights, size=len(edges)),
                              h=rng.integers(-case["hmax"], case["hmax"] + 1, size=n).astype(np.int8),
                              color=color, n_colors=n_colors, b=b, K=K, T=T, Gamma=case["gamma"]))
    return out


def _network_inputs(case, seed):
    """Parameters with every layer in use, standardised features, targets in [0, 1]."""
    rng = np.random.default_rng([GRAPH_SEED, 7, int(seed)])
    p = ptqmc.init_ladder_params(int(seed))
    p[-64 * 128 - 64:] = rng.normal(0.0, 0.1, 64 * 128 + 64).astype(np.float32)
    x = rng.normal(size=(case["batch"], 32)).astype(np.float32)
    level, slope = rng.uniform(0.1, 0.6, (case["batch"], 1)), rng.uniform(0.0, 0.3, (case["batch"], 1))
    q = np.clip(level + slope * (np.arange(64) / 63 - 0.5), 0.0, 1.0).astype(np.float32)
    if case["loss"] == "softmax":
        q = (q / q.sum(1, keepdims=True)).astype(np.float32)
    return p, x, q


def prepare(case, seed):
    if case["kind"] == "network":
        p, x, q = _network_inputs(case, seed)
        return {"case": case, "net": ptqmc.LadderNet(p), "x": torch.from_numpy(x).cuda(),
                "q": torch.from_numpy(q).cuda()}
    s = ptqmc.Sampler(_instances(case, seed), seed, sweeps_per_exchange=case["k"],
                      encoding=ptqmc.PT_BITPACK32 if case["encoding"] == "bitpack" else ptqmc.PT_INT8,
                      flags=ptqmc.PT_FLAG_TAU_CORR if case["tau"] else 0)
    s.run(BURN_IN)
    s.sync()
    return {"case": case, "sampler": s}


# ------------------------------------------------------------------ a pass

def run(state):
    case = state["case"]
    if case["kind"] == "network":
        net = state["net"]
        if case["op"] == "forward":
            return net.forward(state["x"])
        kind = ptqmc.MLP_LOSS_SIGMOID if case["loss"] == "sigmoid" else ptqmc.MLP_LOSS_SOFTMAX
        loss = net.loss_grad(state["x"], state["q"], kind)
        net.adam(1e-3)
        return {"loss": loss, "grads": net.grads, "params": net.params, "m": net.m, "v": net.v}
    s = state["sampler"]
    s.run(case["cycles"])
    obs = [s.observables(n) for n in range(case["instances"])]
    out = {key: np.concatenate([o[key] for o in obs]) for key in KEYS + (("sumCt",) if case["tau"] else ())}
    out["counts"] = np.array([(o["t"], o["e"], o["n_acc"]) for o in obs], dtype=np.int64)
    if case["spins"]:
        out["spins"] = [s.spins(n) for n in range(case["instances"])]
    return out


# ------------------------------------------------------------------ what a pass cannot do without

def _attempts(case):
    return case["k"] * case["cycles"] * sum(n * m * r for _, n, _, _, m, r in _shapes(case))


def work(case):
    if case["kind"] == "network":
        params = 32 * 128 + 128 + 128 * 128 + 128 + 128 * 64 + 64
        weights = 32 * 128 + 128 * 128 + 128 * 64
        b = case["batch"]
        if case["op"] == "forward":
            return {"bytes": 4 * (params + b * 96), "flops": 2 * b * weights}
        # forward, weight gradients and input gradients of the two upper layers; Adam reads
        # and writes parameters and both moments, and the gradients are written
        return {"bytes": 4 * (7 * params + b * 160), "flops": 2 * b * (3 * weights - 32 * 128)}
    spins = ops = rest = 0
    for graph, n, d, _, m, r in _shapes(case):
        d = d or 6
        spins += n * m * r
        # a draw serves four attempts (one when M = 1): ten rounds of four operations; then
        # field, time field, table index, comparison, update
        ops += n * m * r * ((10 if m > 1 else 40) + d / 2 + 5)
        rest += n * d * 4 + r * (13 * 8 + 8)
    state = spins / (8 if case["encoding"] == "bitpack" else 1)
    return {"bytes": 2 * state + rest + (spins if case["spins"] else 0),
            "flops": ops * case["k"] * case["cycles"]}


# ------------------------------------------------------------------ 64-bit values

def exact(case, seed):
    """The network in float64.  A sampler's outputs are whole numbers and compared as such."""
    if case["kind"] != "network":
        return None
    p32, x, q = _network_inputs(case, seed)
    p = torch.from_numpy(p32.astype(np.float64)).requires_grad_(True)
    x, q = torch.from_numpy(x.astype(np.float64)), torch.from_numpy(q.astype(np.float64))
    sizes = [(128, 32), (128,), (128, 128), (128,), (64, 128), (64,)]
    at, parts = 0, []
    for shape in sizes:
        parts.append(p[at:at + math.prod(shape)].reshape(shape))
        at += math.prod(shape)
    w1, b1, w2, b2, w3, b3 = parts
    z = torch.relu(torch.relu(x @ w1.T + b1) @ w2.T + b2) @ w3.T + b3
    if case["op"] == "forward":
        return z.detach()
    if case["loss"] == "sigmoid":
        loss = (torch.nn.functional.softplus(z) - q * z).sum() / case["batch"]
    else:
        loss = -(q * torch.log_softmax(z, 1)).sum() / case["batch"]
    (g,) = torch.autograd.grad(loss, p)
    m, v = 0.1 * g, 0.001 * g * g
    new = p.detach() - 1e-3 * (m / 0.1) / (torch.sqrt(v / 0.001) + 1e-8)
    return {"loss": float(loss), "grads": g, "params": new, "m": m, "v": v}
