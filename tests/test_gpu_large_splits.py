"""Automatic runs (engine 3 by rounds) of LTSs whose iterations split large
blocks, against engine 2, which scans all states in every iteration: the same
partitions and iteration counts as the oracle's, and no slower.  The bound
leaves half as much again and 1 ms for what is not the kernels' (launches,
clocks); the ratio of what it is there to find was 3 to 500."""
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


def backward_chain(n):
    """s -> s - 1: each block loses its leader, all others are split off."""
    return gen.LTS(n, 1, np.arange(1, n), np.zeros(n - 1, int), np.arange(n - 1))


def fat(q, deg, K, copies):
    """few blocks of many states"""
    return gen.planted_quotient(q, deg, K, seed=1, copies_hi=copies)


def lone_leader(n):
    """all states loop, but for the first, which leads to a state of its own"""
    dst = np.arange(n)
    dst[0] = n - 1
    return gen.LTS(n, 2, np.arange(n), (np.arange(n) == n - 1).astype(int), dst)


def pairs(n, bits):
    """states told apart by `bits` pairs of states they lead to: large splits
    by splitters of very many in-transitions"""
    base = n - 2 * bits
    s = np.arange(base)
    src = [np.tile(s, bits), base + np.arange(2 * bits)]
    lab = [np.repeat(np.arange(bits), base), bits + np.arange(2 * bits) % 2]
    dst = [np.concatenate([base + 2 * i + ((s >> i) & 1) for i in range(bits)]), src[1]]
    return gen.LTS(n, bits + 2, *(np.concatenate(x) for x in (src, lab, dst)))


CASES = {
    "backward-chain-1k": lambda: backward_chain(1000),
    "backward-chain-3k": lambda: backward_chain(3000),
    "backward-chain-10k": lambda: backward_chain(10_000),
    "backward-chain-40k": lambda: backward_chain(40_000),
    "fat-10k": lambda: fat(20, 4.0, 3, 1000),
    "fat-30k": lambda: fat(40, 4.0, 3, 1500),
    "fat-200k": lambda: fat(40, 4.0, 3, 10_000),
    "fat-1M": lambda: fat(100, 6.0, 4, 20_000),
    "lone-leader-20k": lambda: lone_leader(20_000),
    "lone-leader-1M": lambda: lone_leader(1_000_000),
    "no-transitions-5M": lambda: gen.LTS(5_000_000, 2, [0], [0], [1]),
    "sink-2M": lambda: gen.LTS(2_000_000, 1, np.arange(1, 2_000_000), np.zeros(1_999_999, int),
                               np.zeros(1_999_999, int)),
    "pairs-20k": lambda: pairs(20_000, 8),
    "pairs-100k": lambda: pairs(100_000, 8),
}


@pytest.fixture(autouse=True)
def cache(monkeypatch, tmp_path_factory):
    monkeypatch.setenv("BISIM_TUNE_CACHE", str(tmp_path_factory.mktemp("tune") / "tune.txt"))


def best_of(h, out, runs=3):
    times = []
    for _ in range(runs):
        t = time.perf_counter()
        _, st = h.run(out)
        times.append((time.perf_counter() - t) * 1e3)
    return min(times), st


@pytest.mark.parametrize("case", sorted(CASES))
def test_large_splits_no_slower_than_scans(B, case):
    L = CASES[case]()
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    out = B.DeviceArray(L.n, np.int32)
    with B.LTS(*dev, L.n, L.K, None) as h:
        h.run(out)
        auto, st = best_of(h, out)
        assert (out.numpy() == ks).all() and st.blocks == nb
        h.set_option(B.OPT_ENGINE, 2)
        scans, ref = best_of(h, out)
        assert st.iterations == ref.iterations
    print(f"[large splits] {case}: {auto:.2f} ms, engine 2 {scans:.2f}", flush=True)
    assert auto < 1.5 * scans + 1


SHAPES = {c: CASES[c] for c in ("backward-chain-1k", "backward-chain-3k", "fat-10k", "fat-30k",
                                "lone-leader-20k", "pairs-20k")}


@pytest.mark.parametrize("lds", [0, 70000, 30000, 2000])
def test_large_splits_in_a_batch(B, lds):
    """In a batch one workgroup carries out all of them, at any LDS budget."""
    insts = [SHAPES[c]() for c in sorted(SHAPES)]
    with B.Batch(insts) as b:
        b.set_option(B.BOPT_LDS_LIMIT, lds)
        b.set_option(B.BOPT_GRID, 4)
        out, its, st = b.run()
        blocks = b.split(out.numpy())
    print(f"[large splits] batch, LDS {lds}: {st['t_alg_ms']:.1f} ms", flush=True)
    for k, L in enumerate(insts):
        ref = oracle.alg3_trace(L.n, L.K, L.src, L.lab, L.dst)
        assert (blocks[k] == ref["block"]).all() and its[k] == ref["iters"], sorted(SHAPES)[k]


# many transitions per state, few iterations: (LTS, algorithm, learned policy)
DENSE = {
    "16k-2M": (lambda: gen.random_lts(16_000, 2_000_000, 1, 1, init_blocks=3), 3, False),
    "16k-8M": (lambda: gen.random_lts(16_000, 8_000_000, 8, 1), 3, False),
    "30k-8M": (lambda: gen.random_lts(30_000, 8_000_000, 1, 1, init_blocks=2), 3, False),
    "100k-10M": (lambda: gen.random_lts(100_000, 10_000_000, 2, 1), 3, False),
    "algorithm-2-16k-2M": (lambda: gen.kripke_uniform(16_000, 2_000_000, 1), 2, False),
    "learned-2k-1M": (lambda: gen.kripke_uniform(2_000, 1_000_000, 1), 3, True),
    "learned-2k-200k-64": (lambda: gen.random_lts(2_000, 200_000, 64, 1), 3, True),
}


@pytest.mark.parametrize("case", sorted(DENSE))
def test_dense_no_slower_than_scans(B, case):
    make, algorithm, learned = DENSE[case]
    L = make()
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst, L.init)
    dev = [None if a is None else B.DeviceArray.from_numpy(a, np.int32)
           for a in (L.src, L.lab, L.dst, L.init)]
    out = B.DeviceArray(L.n, np.int32)
    with B.LTS(*dev[:3], L.n, L.K, dev[3]) as h:
        h.set_option(B.OPT_ALGORITHM, algorithm)
        w = B.MLP(B.POLICY_FEATURES, seed=1) if learned else None
        if learned:
            B.set_splitter_policy(h, B.POLICY_LEARNED, w)
        h.run(out)
        auto, st = best_of(h, out)
        ran = h.run_config()
        assert (out.numpy() == ks).all() and st.blocks == nb
        h.set_option(B.OPT_ENGINE, 2)
        scans, ref = best_of(h, out)
        assert st.iterations == ref.iterations
    print(f"[large splits] {case}: {auto:.2f} ms by {ran}, engine 2 {scans:.2f}", flush=True)
    assert auto < 1.5 * scans + 0.3


def test_many_actions_choose_between_the_engines(B, monkeypatch, tmp_path):
    """States of more than 64 actions go in lock step: from 200,000 states on
    engines 2 and 3 are both timed on the first iterations, once."""
    cache = tmp_path / "tune.txt"
    monkeypatch.setenv("BISIM_TUNE_CACHE", str(cache))
    L = gen.uniform_lts(2000, 3.0, 90, seed=6)
    hub = np.arange(80)  # one state with 80 actions, and others without any
    L = gen.LTS(300_000, 90, np.concatenate([L.src, np.zeros(80, int)]),
                np.concatenate([L.lab, hub]), np.concatenate([L.dst, hub * 97 % L.n]))
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    with B.LTS(*dev, L.n, L.K, None) as h:
        for _ in range(2):
            out, st = h.run()
            assert (out.numpy() == ks).all() and st.blocks == nb
            engine, grid = h.run_config()
            chosen = [x.split() for x in cache.read_text().splitlines()]
            assert len(chosen) == 1 and chosen[0][1:3] == [str(engine), str(grid)]
            assert chosen[0][0].startswith("lts_") and "rounds" not in chosen[0][0]
