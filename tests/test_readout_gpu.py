"""Read-back of spins and observables: whole, in order, at the edges of the device's 16-byte
pieces and of the pinned buffers, and after a resident launch gave up."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

# (N, M, R): one 16-byte piece and less, ragged ends, M = 1 and 2, 33 slots (two word groups),
# and 2 MiB buffers: one exactly full, two, and three with a ragged end
SHAPES = [(2, 2, 2), (5, 1, 3), (5, 6, 3), (16, 8, 33), (7, 1, 65), (64, 512, 64), (67, 1024, 33), (331, 128, 107)]


@pytest.mark.parametrize("encoding", [ptqmc.PT_INT8, ptqmc.PT_BITPACK32])
@pytest.mark.parametrize("N,M,R", SHAPES)
def test_spins_come_back_as_set(N, M, R, encoding):
    print(f"case: spins N={N} M={M} R={R} encoding={encoding}", flush=True)
    rng = np.random.default_rng([N, M, R])
    insts = [W.random_small_instance(rng, N, M, R, d=2, name="a"),
             W.random_small_instance(rng, 9, 8, 3, d=2, name="b")]
    with ptqmc.Sampler(insts, 5, encoding=encoding) as s:
        for n, (shape) in enumerate([(R, M, N), (3, 8, 9)]):
            x = rng.choice(np.array([-1, 1], np.int8), size=shape)
            s.set_spins(n, x)
            assert np.array_equal(s.spins(n), x)
            assert np.array_equal(s.spins(n), x)


@pytest.mark.parametrize("read", ["observables", "spins"])
def test_first_read_after_a_wait_that_gave_up(read):
    """The read that finds the failed launch returns the recovered state."""
    print(f"case: recovery found by {read}", flush=True)
    rng = np.random.default_rng(77)
    inst = W.random_small_instance(rng, 40, 128, 3, d=4, jmax=2, name="blocks")
    flags = ptqmc.PT_FLAG_SLICE_BLOCKS | ptqmc.PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT | ptqmc.PT_FLAG_NO_GRAPH
    ref = oracle.OracleChain(inst, 9, index=0)
    ref.run(4, 2)
    with ptqmc.Sampler([inst], 9, sweeps_per_exchange=4, flags=flags, block_threads=256) as s:
        s.run(2)
        if read == "spins":
            assert np.array_equal(s.spins(0), ref.s)
        else:
            got, want = s.observables(0), ref.observables()
            for k in ("E_cl", "C", "rung_of", "sumE", "sumC2", "acc", "label"):
                assert np.array_equal(np.asarray(got[k]), np.asarray(want[k])), k
        assert s.info()["recoveries"] == 1
