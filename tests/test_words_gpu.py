"""Word tiles (any slice count, M = 1 and 2, large couplings; both encodings) against the
oracle: rows of one to sixteen words with every remainder, quads of replicas with every
remainder, each form of the table index, compiled and run-time degrees, one colour class and
many, and workgroups from the smallest on."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

KEYS = ("E_cl", "C", "rung_of", "replica_of", "acc", "att", "roundtrips", "label", "sumE", "sumC",
        "sumE2", "sumC2", "nup", "ndown")


def batch():
    rng = np.random.default_rng([1004, 41])
    mk = lambda *a, **k: W.random_small_instance(rng, *a, **k)
    lone = W.make_instance(3, np.zeros((0, 2), np.int32), np.zeros(0, np.int8), np.array([1, -1, 1], np.int8),
                           20, [0.5, 1.0, 2.0], 1.0, name="lone")
    return [
        mk(10, 1, 4, d=3, jmax=3), mk(12, 1, 9, d=3, jmax=8), mk(12, 1, 34, d=3, jmax=30),   # M = 1: F <= 20, 63, more
        mk(7, 2, 2, d=2, hmax=0), mk(12, 2, 6, d=3, jmax=100, hmax=50, t_min=5, t_max=50),   # M = 2
        mk(5, 4, 3, d=2, jmax=2, hmax=2), mk(9, 6, 5, d=4, jmax=3), mk(8, 14, 33, d=5),      # part rows
        mk(9, 12, 40, d=4, jmax=2), mk(20, 24, 11, d=8, jmax=2), mk(30, 100, 5, d=4, jmax=9, hmax=4),
        mk(33, 10, 7, d=3, jmax=120, hmax=100, t_min=2.0), mk(12, 4, 6, d=11),               # wide; degree > 8
        mk(13, 8, 5, d=4, jmax=7, hmax=5, relabel=False),                                    # power-of-two rows, F > 20
        mk(64, 126, 70, d=6), lone,
    ]


def check(s, n, ref, what):
    got, want = s.observables(n), ref.observables()
    for key in KEYS:
        assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), f"{what} instance {n}: {key}"
    assert np.array_equal(s.spins(n), ref.s), f"{what} instance {n}: spins"


@pytest.fixture(scope="module")
def refs():
    out = []
    for n, inst in enumerate(batch()):
        r = oracle.OracleChain(inst, 77, index=n)
        r.run(3, 20)
        r.sweep(2)
        out.append(r)
    return out


@pytest.mark.parametrize("encoding", [ptqmc.PT_INT8, ptqmc.PT_BITPACK32])
@pytest.mark.parametrize("shape", [{}, dict(tile_replicas=1), dict(tile_replicas=5, block_threads=192),
                                   dict(block_threads=64), dict(tile_replicas=32, block_threads=256)],
                         ids=lambda s: "-".join(f"{k}{v}" for k, v in s.items()) or "tuned")
def test_word_tiles_match_oracle(refs, encoding, shape):
    print(f"case: word tiles encoding={encoding} {shape}", flush=True)
    with ptqmc.Sampler(batch(), 77, sweeps_per_exchange=3, encoding=encoding, **shape) as s:
        s.run(20)
        s.sweep(2)
        for n, ref in enumerate(refs):
            check(s, n, ref, f"{encoding} {shape}")


@pytest.mark.parametrize("encoding", [ptqmc.PT_INT8, ptqmc.PT_BITPACK32])
def test_word_tiles_graph_replays(refs, encoding):
    """Each replay of the captured cycles against the oracle, with eager calls between them."""
    print(f"case: word tiles, graph replays, encoding={encoding}", flush=True)
    insts = batch()
    refs = [oracle.OracleChain(inst, 5, index=n) for n, inst in enumerate(insts)]
    with ptqmc.Sampler(insts, 5, sweeps_per_exchange=2, encoding=encoding, block_threads=256) as s:
        for replay in range(3):
            s.run(16)
            s.sweep(1)
            for n, ref in enumerate(refs):
                ref.run(2, 16)
                ref.sweep(1)
                check(s, n, ref, f"replay {replay}")
