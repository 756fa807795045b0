"""How long tuning lasts: within the 45 cycles that three timings of each of a byte batch's fifteen
shapes take, whatever shapes there are to try and however a program asks for the cycles."""
import numpy as np
import pytest

import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu


def regular(N, M, R, n=1, jmax=1):
    rng = np.random.default_rng([1004, 71, N, M])
    edges = W.random_regular_graph(N, 6, rng)
    J = np.array([v for v in range(-jmax, jmax + 1) if v], np.int8)
    return [W.make_instance(N, edges, rng.choice(J, size=len(edges)), np.zeros(N, np.int8), M,
                            W.geometric_temperatures(0.2, 3.0, R), 1.0) for _ in range(n)]


BATCHES = {
    "one instance": (lambda: regular(128, 64, 32, jmax=3), ptqmc.PT_INT8),
    "octets on bytes": (lambda: regular(64, 64, 64, n=16), ptqmc.PT_INT8),
    "word tiles": (lambda: regular(51, 20, 24, n=4), ptqmc.PT_INT8),
    "many word tiles": (lambda: regular(51, 100, 64, n=40, jmax=3), ptqmc.PT_INT8),
    "packed": (lambda: regular(64, 64, 40, n=8), ptqmc.PT_BITPACK32),
}


@pytest.mark.parametrize("call", [1, 8, 45])
@pytest.mark.parametrize("batch", BATCHES)
def test_tuned_within_45_cycles(batch, call):
    print(f"case: tuning of {batch}, {call} cycles a call", flush=True)
    make, encoding = BATCHES[batch]
    with ptqmc.Sampler(make(), 5, sweeps_per_exchange=4, encoding=encoding) as s:
        for at in range(0, 45, call):
            s.run(min(call, 45 - at))
        info = s.info()
        assert info["tuned"] == 1 and s.observables(0)["e"] == 45
