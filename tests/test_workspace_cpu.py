"""pt_workspace_bytes of byte batches that could run as octets: the octets' tables (512 bytes a
replica) are in it only where the tuner may choose them, and never for a batch of millions of
replicas."""
import ctypes as C
import os

import numpy as np
import pytest

import workloads as W
from paper_1004_0023_amd import ptqmc

TABLE_BYTES = 512


def nbytes(insts, **options):
    if not os.path.exists(ptqmc.LIB_PATH):
        pytest.skip("library not built")
    recs, keep = ptqmc._records(insts)
    opt = ptqmc._options(1, 1, ptqmc.PT_INT8, 0, options.get("tile_replicas", 0), 0, 0)
    out = C.c_size_t(0)
    ptqmc._check(ptqmc.lib().pt_workspace_bytes(C.cast(recs, C.c_void_p), len(insts), C.byref(opt), C.byref(out)))
    return out.value


def batch(n, R):
    """n pairs of coupled spins, 8 slices, R replicas each."""
    one = W.make_instance(2, np.array([[0, 1]], np.int32), np.ones(1, np.int8), np.zeros(2, np.int8), 8, [1.0, 2.0], 1.0)
    T = np.linspace(1.0, 2.0, R)
    b, K = W.st_rungs(T, 1.0, 8)
    return [one.with_ladder(b, K, T) for _ in range(n)]


@pytest.mark.parametrize("n,R", [(1, 32), (14, 65), (2, 1_060_000)], ids=["one", "too few octets", "too many replicas"])
def test_no_octet_tables_without_octets(n, R):
    insts = batch(n, R)
    assert nbytes(insts) == nbytes(insts, tile_replicas=1)


def test_octet_tables_where_octets_are_offered():
    insts = batch(16, 64)  # 128 octets
    extra = nbytes(insts) - nbytes(insts, tile_replicas=1)
    assert 16 * 64 * TABLE_BYTES <= extra <= 16 * 64 * TABLE_BYTES + 16384
