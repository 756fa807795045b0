"""Octet kernels on instances whose sites have different degrees, against the oracle: rows padded
by none to all of their entries, with and without fields, in whole octets and in slice blocks
(resident, and launched per parity)."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

KEYS = ("E_cl", "C", "rung_of", "replica_of", "acc", "att", "roundtrips", "label", "sumE", "sumC",
        "sumE2", "sumC2", "nup", "ndown")


def instance(rng, edges, n, m, r, hmax):
    edges = np.array(sorted({(min(a, b), max(a, b)) for a, b in edges}), np.int32)
    J = rng.choice(np.array([-1, 1], np.int8), size=len(edges))
    h = rng.integers(-hmax, hmax + 1, size=n).astype(np.int8)
    return W.make_instance(n, edges, J, h, m, W.geometric_temperatures(0.3, 3.0, r), 1.0)


def open_lattice(lx, ly, lz):
    at = lambda x, y, z: x + lx * (y + ly * z)
    return [(at(x, y, z), at(x + dx, y + dy, z + dz)) for z in range(lz) for y in range(ly) for x in range(lx)
            for dx, dy, dz in ((1, 0, 0), (0, 1, 0), (0, 0, 1)) if x + dx < lx and y + dy < ly and z + dz < lz]


def batch():
    rng = np.random.default_rng([1004, 42])
    star = lambda d: [(0, k) for k in range(1, d + 1)]
    out = [instance(rng, star(d), 10, 8, 9, hmax) for d in range(1, 9) for hmax in (0, 1)]  # hubs, leaves, lone sites
    out.append(instance(rng, open_lattice(3, 4, 5), 60, 64, 33, 1))
    out.append(instance(rng, [(k, k + 1) for k in range(39)], 40, 16, 8, 0))                # a path
    pairs = rng.integers(0, 50, (90, 2))
    deg, edges = np.zeros(50, int), set()
    for a, b in pairs:
        if a != b and deg[a] < 8 and deg[b] < 8 and (min(a, b), max(a, b)) not in edges:
            edges.add((min(a, b), max(a, b)))
            deg[a] += 1
            deg[b] += 1
    out.append(instance(rng, edges, 50, 32, 20, 1))
    return out


def check(s, n, ref):
    got, want = s.observables(n), ref.observables()
    for key in KEYS:
        assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), f"instance {n}: {key}"
    assert np.array_equal(s.spins(n), ref.s), f"instance {n}: spins"


@pytest.mark.parametrize("threads", [64, 256, 1024])
def test_whole_octets(threads):
    print(f"case: octets of mixed degrees, {threads} threads", flush=True)
    insts = batch()
    with ptqmc.Sampler(insts, 8, sweeps_per_exchange=3, encoding=ptqmc.PT_BITPACK32, block_threads=threads) as s:
        info = s.info()
        assert info["oct_blocks"] == 0 and info["class_launches"] == 0 and info["n_tiles"] == 0
        s.run(18)
        s.sweep(2)
        for n, inst in enumerate(insts):
            ref = oracle.OracleChain(inst, 8, index=n)
            ref.run(3, 18)
            ref.sweep(2)
            check(s, n, ref)


@pytest.mark.parametrize("per_sweep", [False, True])
def test_slice_blocks(per_sweep):
    print(f"case: octet slice blocks of mixed degrees, per sweep {per_sweep}", flush=True)
    rng = np.random.default_rng([1004, 43])
    inst = instance(rng, open_lattice(8, 8, 9), 576, 128, 10, 1)
    with ptqmc.Sampler([inst], 8, sweeps_per_exchange=3, encoding=ptqmc.PT_BITPACK32,
                       flags=ptqmc.PT_FLAG_BLOCK_LAUNCH_PER_SWEEP if per_sweep else 0) as s:
        assert s.info()["oct_blocks"] > 0 and s.info()["oct_resident"] == (0 if per_sweep else 1)
        s.run(3)
        s.sweep(2)
        ref = oracle.OracleChain(inst, 8, index=0)
        ref.run(3, 3)
        ref.sweep(2)
        check(s, 0, ref)
