"""States of very many in-transitions (sinks): results equal the oracle's, and
what is laid out once per handle is spread over transitions, not targets.  One
lane that walks a million transitions takes 0.4 s; the bounds leave
the layout 50 ms, a hundred times what its bytes take."""
import time

import numpy as np
import pytest

import oracle
from paper_2105_11788_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2105_11788_amd import bisim
    return bisim


def sink(n, actions):
    """Every state but the sink has a transition of each action to it."""
    src = np.repeat(np.arange(1, n), actions)
    return gen.LTS(n, actions, src, np.tile(np.arange(actions), n - 1), np.zeros(src.size, int))


def timed(f):
    t = time.perf_counter()
    r = f()
    return r, (time.perf_counter() - t) * 1e3


def first_and_next(B, L, learned=False):
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    out = B.DeviceArray(L.n, np.int32)
    with B.LTS(*dev, L.n, L.K, None) as h:
        w = B.MLP(B.POLICY_FEATURES, seed=1) if learned else None
        if learned:
            B.set_splitter_policy(h, B.POLICY_LEARNED, w)
        (_, st), first = timed(lambda: h.run(out))
        _, later = timed(lambda: h.run(out))
        return out.numpy(), st, first, later


def test_sink_first_run(B):
    first_and_next(B, sink(100, 2))  # (the kernels are loaded)
    first_and_next(B, sink(100, 2), learned=True)
    L = sink(100_001, 10)
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    for learned in (False, True):
        got, st, first, later = first_and_next(B, L, learned)
        print(f"[sink] learned {learned}: first {first:.1f} ms, next {later:.1f}", flush=True)
        assert (got == ks).all() and st.blocks == nb
        assert first < later + 50


def test_sink_batch_load(B):
    L = sink(100_001, 10)
    small = gen.kripke_uniform(100, 500, seed=1)
    B.Batch([small]).close()
    with B.Batch([L, small]) as b:
        b.set_option(B.BOPT_GRID, 2)
        out, its, st = b.run()
        got = b.split(out.numpy())
    print(f"[sink] batch load {st['t_pre_ms']:.1f} ms", flush=True)
    assert (got[0] == oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)[0]).all()
    assert st["t_pre_ms"] < 100  # (23 ms of them the load's atomics at the sink)


@pytest.mark.parametrize("n,actions,loop", [(100_001, 10, False), (100_000, 10, True)])
def test_sink_marked_by_the_grid(B, n, actions, loop):
    """One state's in-transitions are spread over the grid, so a run is no
    slower than engine 2's, whose wave takes them 64 at a time."""
    L = sink(n, actions)
    if loop:  # the sink has the others' actions: one block
        L = gen.LTS(n, actions, *(np.concatenate([x, y]) for x, y in (
            (L.src, np.zeros(actions, int)), (L.lab, np.arange(actions)),
            (L.dst, np.zeros(actions, int)))))
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    out = B.DeviceArray(L.n, np.int32)
    best = {}
    with B.LTS(*dev, L.n, L.K, None) as h:
        for engine in (3, 2):
            h.set_option(B.OPT_ENGINE, engine)
            h.run(out)
            runs = [timed(lambda: h.run(out)) for _ in range(3)]
            best[engine] = min(ms for _, ms in runs)
            st = runs[0][0][1]
            assert st.blocks == (1 if loop else 2) and st.iterations == (2 if loop else 3)
            assert (out.numpy() == np.minimum(np.arange(n), 0 if loop else 1)).all()
    print(f"[sink] {n} states, {L.m} transitions: engine 3 {best[3]:.2f} ms, 2 {best[2]:.2f}",
          flush=True)
    assert best[3] < 1.5 * best[2] + 1


def test_sink_signature_rounds(B):
    """The targets of the transitions are written by all waves: one lane takes
    25 ns for each of a sink's, 0.25 s here; the rounds' sorts and hash tables
    are a few passes over 10M transitions, below 10 ms at a tenth of the
    memory's rate."""
    L = sink(1_000_001, 10)
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    out = B.DeviceArray(L.n, np.int32)
    with B.LTS(*dev, L.n, L.K, None) as h:
        h.set_option(B.OPT_ALGORITHM, B.ALGORITHM_SIGNATURE)
        h.run(out)
        runs = [timed(lambda: h.run(out))[1] for _ in range(3)]
    print(f"[sink] signature rounds {min(runs):.1f} ms", flush=True)
    assert (out.numpy() == np.minimum(np.arange(L.n), 1)).all()
    assert min(runs) < 100
