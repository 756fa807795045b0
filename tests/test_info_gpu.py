"""The launch record of routes that are not byte tiles."""
import numpy as np
import pytest

import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("encoding", [ptqmc.PT_INT8, ptqmc.PT_BITPACK32])
def test_word_tiles_report_their_lds(encoding):
    print(f"case: launch record of word tiles, encoding {encoding}", flush=True)
    inst = W.random_small_instance(np.random.default_rng(3), 30, 12, 9, d=4, jmax=3)
    with ptqmc.Sampler([inst], 1, encoding=encoding, tile_replicas=3, block_threads=256) as s:
        info = s.info()
    assert info["n_tiles"] == 3 and info["max_tile_replicas"] == 3
    assert 3 * 30 * 12 <= info["lds_bytes"] <= 163840


def test_octets_on_bytes_report_no_byte_tiles():
    print("case: launch record of octets on bytes", flush=True)
    rng = np.random.default_rng(4)
    edges = W.random_regular_graph(256, 6, rng)
    insts = [W.make_instance(256, edges, rng.choice(np.array([-1, 1], np.int8), size=len(edges)),
                             np.zeros(256, np.int8), 64, W.geometric_temperatures(0.2, 3.0, 64), 1.0)
             for _ in range(64)]
    with ptqmc.Sampler(insts, 1, sweeps_per_exchange=10) as s:
        s.run(48)
        info = s.info()
    assert info["tuned"] == 1
    if info["oct_tiles"] == 0:
        pytest.skip("the tuner kept the byte tiles")
    assert info["oct_tiles"] == 512
    assert info["n_tiles"] == 0 and info["sweep_groups"] == 0 and 256 * 64 <= info["lds_bytes"] <= 163840
