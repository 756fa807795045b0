"""Calls that meet a launch that gave up a wait, before any synchronisation has seen it: the
state they leave, write out or return is the chain's, or the call says that it is not."""
import numpy as np
import pytest

import oracle
import workloads as W
from paper_1004_0023_amd import ptqmc

pytestmark = pytest.mark.gpu

KEYS = ("E_cl", "C", "rung_of", "replica_of", "acc", "att", "roundtrips", "label", "sumE", "sumC",
        "sumE2", "sumC2", "nup", "ndown")
SEED, K = 21, 2


def words(rng):
    mk = lambda *a, **k: W.random_small_instance(rng, *a, **k)
    return [mk(12, 6, 9, d=3, jmax=8), mk(10, 1, 70, d=3, jmax=3), mk(9, 12, 67, d=4)]


def fast(rng):
    return [W.random_small_instance(rng, 12, 64, 8), W.random_small_instance(rng, 8, 32, 66, d=4)]


def blocks(rng):
    edges = W.cubic_lattice(6, 6, 6)
    return [W.make_instance(216, edges, rng.choice(np.array([-1, 1], np.int8), size=len(edges)),
                            np.zeros(216, np.int8), 512, W.geometric_temperatures(0.3, 3.0, R), 1.0) for R in (3, 13)]


# routes whose tiles wait for each other, with fixed shapes: the first run gives up its waits
ROUTES = {
    "words-bytes": (words, dict(block_threads=256)),
    "words-packed": (words, dict(block_threads=256, encoding=ptqmc.PT_BITPACK32)),
    "fast": (fast, dict(tile_replicas=4, block_threads=512)),
    "octet-blocks": (blocks, dict(encoding=ptqmc.PT_BITPACK32)),
}


def build(route):
    make, shape = ROUTES[route]
    return make(np.random.default_rng([1004, 61])), shape


def chains(insts, cycles):
    refs = [oracle.OracleChain(inst, SEED, index=n) for n, inst in enumerate(insts)]
    for r in refs:
        r.run(K, cycles)
    return refs


def gives_up(insts, shape, **more):
    return ptqmc.Sampler(insts, SEED, sweeps_per_exchange=K, flags=ptqmc.PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT, **shape,
                         **more)


def check(s, refs, what):
    for n, ref in enumerate(refs):
        got, want = s.observables(n), ref.observables()
        for key in KEYS:
            assert np.array_equal(np.asarray(got[key]), np.asarray(want[key])), f"{what} instance {n}: {key}"
        assert np.array_equal(s.spins(n), ref.s), f"{what} instance {n}: spins"


@pytest.mark.parametrize("route", ROUTES)
def test_set_spins(route):
    """Spins set in one instance: the others are the chain's, and so is what follows."""
    print(f"case: spins set after a wait that gave up, {route}", flush=True)
    insts, shape = build(route)
    refs = chains(insts, 6)
    x = np.random.default_rng(5).choice(np.array([-1, 1], np.int8), size=refs[1].s.shape)
    refs[1].s[...] = x
    refs[1].E[...], refs[1].C[...] = refs[1].energies()
    with gives_up(insts, shape) as s:
        s.run(6)
        s.set_spins(1, x)
        check(s, refs, "set")
        assert s.info()["recoveries"] == 1
        s.run(3)
        for r in refs:
            r.run(K, 3)
        check(s, refs, "after")


@pytest.mark.parametrize("route", ROUTES)
def test_save(route):
    """The checkpoint that the failed launch's recovery precedes holds the chain's state."""
    print(f"case: checkpoint after a wait that gave up, {route}", flush=True)
    insts, shape = build(route)
    refs = chains(insts, 6)
    with gives_up(insts, shape) as s:
        s.run(6)
        blob = s.save()
        assert s.info()["recoveries"] == 1
    with ptqmc.Sampler(insts, SEED, sweeps_per_exchange=K, **shape) as s:
        s.load(blob)
        check(s, refs, "loaded")


@pytest.mark.parametrize("route", ROUTES)
def test_replays_of_a_callers_graph_are_not_dropped(route):
    """A recovery cannot know of replays: a wait that gave up before the capture (or, of resident
    slice blocks, in a replay) is an error then, never a state without them."""
    import torch
    print(f"case: a caller's graph after a wait that gave up, {route}", flush=True)
    insts, shape = build(route)
    stream = torch.cuda.Stream()
    with gives_up(insts, shape, stream=stream) as s:
        if route != "octet-blocks":
            s.run(20)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            s.run(4)
        for _ in range(3):
            with torch.cuda.stream(stream):
                graph.replay()
        with pytest.raises(ptqmc.PTError) as e:
            s.observables(0)
        assert e.value.code == ptqmc.PT_ESTATE and s.info()["recoveries"] == 0


@pytest.mark.parametrize("seen", [False, True], ids=["pending", "failed"])
@pytest.mark.parametrize("route", ["words-bytes", "words-packed", "fast"])
def test_load(route, seen):
    """A checkpoint loaded over such a launch's state, whether or not its failure was reported
    first, is the state the next cycles start from."""
    import torch
    print(f"case: checkpoint loaded after a wait that gave up, {route}, seen {seen}", flush=True)
    insts, shape = build(route)
    refs = chains(insts, 4)
    with ptqmc.Sampler(insts, SEED, sweeps_per_exchange=K, **shape) as s:
        s.run(4)
        blob = s.save()
    stream = torch.cuda.Stream()
    with gives_up(insts, shape, stream=stream) as s:
        s.run(300)
        if seen:
            with torch.cuda.graph(torch.cuda.CUDAGraph(), stream=stream):
                s.run(1)
            with pytest.raises(ptqmc.PTError):
                s.sync()
        s.load(blob)
        for _ in range(3):
            s.run(1)  # the exchange step in the launch, by the tiles' counts
        for r in refs:
            r.run(K, 3)
        check(s, refs, "continued")
        assert s.info()["recoveries"] == 0


def test_tuning_onto_a_shape_that_waits_for_nothing():
    """200 whole octets, where the tuner also times 50 resident word tiles: a wait that one of them
    gives up is recovered from there and then, although octets win and nothing can later."""
    print("case: a timed shape gave up a wait, another one won", flush=True)
    rng = np.random.default_rng([1004, 62])
    edges = W.random_regular_graph(64, 6, rng)
    insts = [W.make_instance(64, edges, rng.choice(np.array([-1, 1], np.int8), size=len(edges)),
                             np.zeros(64, np.int8), 64, W.geometric_temperatures(0.2, 3.0, 64), 1.0)
             for _ in range(25)]
    packed = dict(sweeps_per_exchange=10, encoding=ptqmc.PT_BITPACK32, tile_replicas=32)
    with ptqmc.Sampler(insts, SEED, block_threads=512, **packed) as a, \
            ptqmc.Sampler(insts, SEED, flags=ptqmc.PT_FLAG_TEST_BLOCK_WAIT_TIMEOUT, **packed) as s:
        a.run(100)
        a.sweep(3)
        s.run(70)
        s.run(30)
        s.sweep(3)
        s.sync()
        info = s.info()
        assert info["tuned"] == 1 and info["oct_tiles"] == 200 and info["recoveries"] == 1, info
        assert a.info()["multi_launches"] == 0
        for n in range(len(insts)):
            got, want = s.observables(n), a.observables(n)
            for key in KEYS:
                assert np.array_equal(got[key], want[key]), f"instance {n}: {key}"
            assert np.array_equal(s.spins(n), a.spins(n)), f"instance {n}: spins"


@pytest.mark.parametrize("k,calls,shape", [(2, (30, 50, 300, 100), {}),
                                           (200, (40, 1000, 1000), dict(tile_replicas=1, block_threads=1024))],
                         ids=["tuned", "full"])
def test_two_contexts_at_work(k, calls, shape):
    """Two contexts, a thread each; in the second case 210 resident tiles each, one of which
    fills a compute unit, for longer than a wait lasts: whichever gives up a wait, both chains
    are those of contexts alone."""
    import threading
    print(f"case: two contexts at work at the same time, {shape}", flush=True)
    rng = np.random.default_rng([1004, 63])
    batches = [[W.random_small_instance(rng, 65, 20, 70, d=4, jmax=3) for _ in range(3)] for _ in range(2)]
    alone = []
    for insts in batches:
        with ptqmc.Sampler(insts, SEED, sweeps_per_exchange=k, block_threads=256, flags=ptqmc.PT_FLAG_NO_GRAPH) as a:
            a.run(sum(calls))
            alone.append([(a.observables(n), a.spins(n)) for n in range(3)])
    failed = []

    def work(b):
        try:
            with ptqmc.Sampler(batches[b], SEED, sweeps_per_exchange=k, **shape) as s:
                for cycles in calls:
                    s.run(cycles)
                for n, (want, spins) in enumerate(alone[b]):
                    got = s.observables(n)
                    for key in KEYS:
                        assert np.array_equal(got[key], want[key]), f"context {b} instance {n}: {key}"
                    assert np.array_equal(s.spins(n), spins), f"context {b} instance {n}: spins"
                print(f"context {b}: recoveries {s.info()['recoveries']}", flush=True)
        except Exception as e:
            failed.append(e)

    threads = [threading.Thread(target=work, args=(b,)) for b in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed, failed


def test_uneven_rings_of_a_long_cycle():
    """66 octets as rings of 4 blocks, some of which share units: their instance's exchange step
    waits for the slowest ring's 2000 sweeps without giving up."""
    print("case: octet slice blocks, uneven rings, 2000 sweeps a cycle", flush=True)
    rng = np.random.default_rng([1004, 64])
    N, M, R = 2600, 32, 528
    edges = np.array(sorted({tuple(sorted((i, (i + d) % N))) for i in range(N) for d in (1, 5)}), np.int32)
    T = W.geometric_temperatures(0.3, 3.0, R)
    b, Kr = W.st_rungs(T, 1.0, M)
    inst = W.Instance(N=N, M=M, R=R, edges=edges, J=rng.choice(np.array([-1, 1], np.int8), size=len(edges)),
                      h=np.zeros(N, np.int8), color=(np.arange(N) % 13).astype(np.uint8), n_colors=13, b=b, K=Kr,
                      T=T, Gamma=1.0)
    packed = dict(sweeps_per_exchange=2000, encoding=ptqmc.PT_BITPACK32)
    with ptqmc.Sampler([inst], SEED, **packed) as s, \
            ptqmc.Sampler([inst], SEED, flags=ptqmc.PT_FLAG_BLOCK_LAUNCH_PER_SWEEP, **packed) as a:
        assert s.info()["oct_blocks"] == 264 and s.info()["oct_resident"] == 1
        s.run(2)
        got = s.observables(0)
        assert s.info()["multi_cycles"] == 2 and s.info()["recoveries"] == 0
        a.run(2)
        want = a.observables(0)
        for key in KEYS:
            assert np.array_equal(got[key], want[key]), key


@pytest.mark.parametrize("first", [0, 5])
@pytest.mark.parametrize("route", ["words-packed", "words-bytes", "fast"])
def test_a_capture_before_tuning_has_ended(route, first):
    """A call captured as the first one, or while shapes are still timed: every replay is its
    cycles, and so are the calls between."""
    import torch
    print(f"case: a caller's capture while shapes are timed, {route} after {first}", flush=True)
    insts, shape = build(route)
    refs = chains(insts, first)
    stream = torch.cuda.Stream()
    with ptqmc.Sampler(insts, SEED, sweeps_per_exchange=K, encoding=shape.get("encoding", ptqmc.PT_INT8),
                       stream=stream) as s:
        s.run(first)
        s.sync()
        assert s.info()["tuned"] == 0
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            s.run(4)
        for replay in range(3):
            with torch.cuda.stream(stream):
                graph.replay()
            s.run(21)
            for r in refs:
                r.run(K, 25)
            check(s, refs, f"replay {replay}")
