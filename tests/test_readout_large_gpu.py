"""Observables of instances with more replicas than the pinned read-back buffer holds."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

KEYS = ("E_cl", "C", "rung_of", "replica_of", "acc", "att", "roundtrips", "label", "sumE", "sumC",
        "sumE2", "sumC2", "nup", "ndown", "t", "e", "n_acc", "sumCt")


def instance(N, M, R):
    edges = np.array([[i, i + 1] for i in range(N - 1)], np.int32).reshape(-1, 2)
    one = W.make_instance(N, edges, np.ones(len(edges), np.int8), np.full(N, N % 2, np.int8), M, [1.0, 2.0], 1.0)
    T = np.linspace(1.0, 2.0, R)
    b, K = W.st_rungs(T, 1.0, M)
    return one.with_ladder(b, K, T)


def test_observables_of_either_route():
    """The largest instance of the buffer and the first beyond it, in one batch with correlations."""
    print("case: read-back of 32768 and 32769 replicas", flush=True)
    insts = [instance(3, 4, 32769), instance(2, 2, 32768)]
    refs = [oracle.OracleChain(inst, 3, index=n) for n, inst in enumerate(insts)]
    with ptqmc.Sampler(insts, 3, sweeps_per_exchange=2, flags=ptqmc.PT_FLAG_TAU_CORR) as s:
        s.run(1)
        for n, ref in enumerate(refs):
            ref.run(2, 1)
            got, want = s.observables(n), ref.observables()
            for key in KEYS:
                assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), f"instance {n}: {key}"


def test_observables_of_millions_of_replicas():
    """164 bytes a replica pass 2^31 at 13.1 million: accepted, and read back whole."""
    print("case: read-back of 13.2 million replicas", flush=True)
    R = 13_200_000
    with ptqmc.Sampler([instance(1, 1, R)], 3, tile_replicas=64, block_threads=256) as s:
        obs = s.observables(0)
    assert np.array_equal(obs["rung_of"], np.arange(R, dtype=np.int32))
    assert np.array_equal(np.abs(obs["E_cl"]), np.ones(R)) and obs["label"][0] == 1 and not obs["label"][1:].any()
