"""Packed instances that octets or word tiles could take and launches per colour class run faster:
which route a batch gets, and the chain of batches that mix them."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

KEYS = ("E_cl", "C", "rung_of", "replica_of", "acc", "att", "roundtrips", "label", "sumE", "sumC",
        "sumE2", "sumC2", "nup", "ndown")


def instance(edges, n, M, R, jmax):
    rng = np.random.default_rng([1004, 81, n, M, R])
    J = np.array([v for v in range(-jmax, jmax + 1) if v], np.int8)
    return W.make_instance(n, edges, rng.choice(J, size=len(edges)), np.zeros(n, np.int8), M,
                           W.geometric_temperatures(0.3, 3.0, R), 1.0)


def open_lattice(l, M, R):
    at = lambda x, y, z: x + l * (y + l * z)
    edges = [(at(x, y, z), at(x + dx, y + dy, z + dz)) for z in range(l) for y in range(l) for x in range(l)
             for dx, dy, dz in ((1, 0, 0), (0, 1, 0), (0, 0, 1)) if x + dx < l and y + dy < l and z + dz < l]
    return instance(np.array(edges, np.int32), l ** 3, M, R, 1)


def cubic(l, M, R, jmax=3):
    return instance(W.cubic_lattice(l, l, l), l ** 3, M, R, jmax)


def regular(n, M, R, jmax=3):
    return instance(W.random_regular_graph(n, 6, np.random.default_rng(n)), n, M, R, jmax)


def lone_sites(n, M, R):
    return instance(np.zeros((0, 2), np.int32), n, M, R, 1)


ROUTES = {
    # octet slice blocks of several degrees: short sweeps, long ones but enough blocks, too few, too many
    "blocks short": (lambda: [open_lattice(10, 128, 8)], "octets"),
    "blocks enough": (lambda: [open_lattice(16, 64, 64)], "octets"),
    "blocks few": (lambda: [open_lattice(16, 64, 56)], "classes"),
    "blocks not resident": (lambda: [open_lattice(12, 128, 256)], "classes"),
    "blocks of one degree": (lambda: [cubic(16, 32, 8, 1)], "octets"),
    # beside an instance that only launches per class take
    "with classes, octet": (lambda: [cubic(20, 8, 3), open_lattice(7, 64, 8)], "classes"),
    "with classes, words": (lambda: [cubic(20, 8, 3), cubic(4, 64, 8)], "classes"),
    "with classes, many words": (lambda: [cubic(20, 8, 3)] + [cubic(4, 64, 64) for _ in range(17)], "both"),
    "with classes, more classes": (lambda: [cubic(20, 8, 3), regular(128, 64, 8)], "both"),
    # alone
    "lone large": (lambda: [cubic(8, 256, 4)], "classes"),
    "lone large, more replicas": (lambda: [cubic(8, 256, 5)], "words"),
    "lone uncoupled": (lambda: [lone_sites(300, 400, 8)], "classes"),
    "lone small": (lambda: [cubic(8, 128, 2)], "words"),
}


@pytest.mark.parametrize("batch", ROUTES)
def test_route(batch):
    print(f"case: packed route, {batch}", flush=True)
    build, route = ROUTES[batch]
    with ptqmc.Sampler(build(), 2, encoding=ptqmc.PT_BITPACK32) as s:
        info = s.info()
    got = (info["oct_tiles"] + info["oct_blocks"] > 0, info["n_tiles"] > 0, info["class_launches"] > 0)
    assert got == {"octets": (True, False, False), "words": (False, True, False), "classes": (False, False, True),
                   "both": (False, True, True)}[route], (got, info)


@pytest.mark.parametrize("batch", ["with classes, octet", "with classes, words", "with classes, more classes",
                                   "lone uncoupled"])
def test_matches_oracle(batch):
    print(f"case: packed route against the oracle, {batch}", flush=True)
    insts = ROUTES[batch][0]()
    refs = [oracle.OracleChain(inst, 2, index=n) for n, inst in enumerate(insts)]
    with ptqmc.Sampler(insts, 2, sweeps_per_exchange=2, encoding=ptqmc.PT_BITPACK32) as s:
        s.run(18)
        s.sweep(1)
        for n, ref in enumerate(refs):
            ref.run(2, 18)
            ref.sweep(1)
            got, want = s.observables(n), ref.observables()
            for key in KEYS:
                assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), f"instance {n}: {key}"
            assert np.array_equal(s.spins(n), ref.s), f"instance {n}: spins"
