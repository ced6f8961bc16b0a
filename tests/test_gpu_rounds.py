"""GPU parity of the rounds (engine 3 without a trace, and the automatic
engine): splitters that split nothing are decided ahead of their turn, and
block ids, block counts and iteration counts equal the lock-step oracle's.
Whole numbers: no tolerance."""
import numpy as np
import pytest

import oracle
from paper_2105_11788_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2105_11788_amd import bisim
    bisim.load_library()
    assert bisim.device_count() > 0, "GPU tests need a GPU"
    return bisim


def permuted(L, seed):
    p = np.random.default_rng(seed).permutation(L.n)
    init = None
    if L.init is not None:
        init = np.empty(L.n, np.int32)
        init[p] = p[L.init]
    return gen.LTS(L.n, L.K, p[L.src], L.lab, p[L.dst], init, name=L.name)


def run(B, L, engine, algorithm=3):
    t = lambda a: None if a is None else B.DeviceArray.from_numpy(a, np.int32)
    with B.LTS(t(L.src), t(L.lab), t(L.dst), L.n, L.K, t(L.init)) as h:
        h.set_option(B.OPT_ENGINE, engine)
        if algorithm != 3:
            h.set_option(B.OPT_ALGORITHM, algorithm)
        out = []
        for _ in range(2):  # a handle runs again
            blk, st = h.run()
            out.append((blk.numpy(), st.iterations, st.blocks))
        return out, h.run_config()[0]


def check(B, L, algorithm=3, engines=(0, 3)):
    ref = oracle.alg3_trace(L.n, L.K, L.src, L.lab, L.dst, L.init, variant=algorithm)
    nb = len(np.unique(ref["block"]))
    for e in engines:
        got, ran = run(B, L, e, algorithm)
        assert ran == 3, (L.name, e)
        for blk, its, blocks in got:
            assert (blk == ref["block"]).all(), (L.name, e)
            assert its == ref["iters"] and blocks == nb, (L.name, e, its, ref["iters"])


CASES = {
    # words of the label bitmaps and one state
    "n1": lambda: gen.random_lts(1, 3, 2, 1),
    "n63": lambda: gen.random_lts(63, 200, 3, 2),
    "n64": lambda: gen.random_lts(64, 250, 3, 3),
    "n65": lambda: gen.random_lts(65, 250, 2, 4, init_blocks=3),
    "no-transitions": lambda: gen.random_lts(70, 0, 2, 5, init_blocks=4),
    "kripke": lambda: gen.kripke_uniform(1000, 5000, seed=2),
    "uniform": lambda: gen.uniform_lts(4500, 6.0, 5, 7),
    # marks of 33..64 actions take 64-bit words
    "wide-marks": lambda: gen.random_lts(900, 20000, 60, 8),
    "zipf": lambda: gen.uniform_zipf(3000, 12000, 64, seed=9),
    "product": lambda: permuted(gen.sync_product(3, 13, seed=3), 1),
    # splits of hundreds and thousands of states, and whole-LTS splitters:
    # more members than a workgroup's threads, marks in LDS
    "chain": lambda: permuted(gen.chain_tail(3000), 2),
    "chain-in-order": lambda: gen.chain_tail(2100),
    "fan-out": lambda: permuted(gen.fan_out(1500), 3),
    "planted-2-actions": lambda: gen.planted_quotient(150, 6.0, 2, seed=5),
    # a state with thousands of in-transitions
    "hub": lambda: gen.LTS(2500, 3, np.arange(5000) % 2500, np.arange(5000) * 7 % 3,
                           np.where(np.arange(5000) % 3 == 0, 5, np.arange(5000) * 13 % 2500)),
}


@pytest.mark.parametrize("case", sorted(CASES))
def test_rounds_match_lock_step(B, case):
    check(B, CASES[case]())


@pytest.mark.parametrize("n,actions", [(16384, 8), (16385, 8), (20000, 40)])
def test_rounds_setup_border(B, n, actions):
    """The workgroup builds the member lists itself up to 16384 states."""
    check(B, gen.planted_quotient(int(n / 20.5), 5.0, actions, seed=n), engines=(3,))
    L = gen.uniform_zipf(n, 2 * n, actions, seed=4)
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    got, _ = run(B, L, 3)
    assert all((blk == ks).all() and blocks == nb for blk, _, blocks in got)
    assert got[0][1] == got[1][1]


@pytest.mark.parametrize("n,actions", [(120_000, 2), (400_000, 3)])
def test_rounds_leave_large_splitters_to_the_grid(B, n, actions):
    """Mark words beyond LDS: large splitters are carried out grid-wide, with
    the label bitmaps in LDS and (400k) in global memory.  The lock-step
    engine gives the iteration count."""
    L = gen.planted_quotient(int(n / 20.5), 4.0, actions, seed=11)
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    ref, _ = run(B, L, 2)
    got, ran = run(B, L, 3)
    assert ran == 3
    for blk, its, blocks in got:
        assert (blk == ks).all() and blocks == nb and its == ref[0][1]


TRACKED = {
    # large splitters that lose single states between their iterations
    "uniform-2-actions": lambda: gen.uniform_lts(30000, 3.0, 2, 5),
    "uniform-1-action-wide": lambda: gen.uniform_lts(9000, 12.0, 1, 6),
    "chain": lambda: permuted(gen.chain_tail(40000), 7),
    "fan-out": lambda: permuted(gen.fan_out(9000), 8),
    "planted-2-actions": lambda: gen.planted_quotient(2500, 5.0, 2, seed=9),
    # tracking starts after some whole blocks were marked: mark words in LDS
    # (and stops again), and beyond LDS with few transitions
    "chain-in-lds": lambda: permuted(gen.chain_tail(12000), 11),
    "uniform-in-lds": lambda: gen.uniform_lts(14000, 5.0, 1, 12),
    "uniform-few-transitions": lambda: gen.uniform_lts(28000, 2.2, 1, 13),
    # 64-bit marks: the mark words of 20k states do not fit LDS
    "wide-marks": lambda: gen.uniform_zipf(20000, 60000, 40, seed=10),
}


@pytest.mark.parametrize("case", sorted(TRACKED))
def test_rounds_track_large_splitters(B, case):
    """Splitters of thousands of in-transitions are re-examined through the
    states they lost; the lock-step engine gives the iteration count."""
    L = TRACKED[case]()
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    ref, _ = run(B, L, 2)
    got, _ = run(B, L, 3)
    with B.Batch([L, L]) as b:
        b.set_option(B.BOPT_GRID, 2)
        out, its, _ = b.run()
        both = b.split(out.numpy())
    for blk, n_it in [(x, i) for x, i, _ in got] + list(zip(both, its)):
        assert (blk == ks).all() and n_it == ref[0][1]
    assert got[0][2] == nb


# more blocks of hundreds of in-transitions than labels are tracked at a time
MANY_LARGE = {
    "propositions": lambda: gen.random_lts(50000, 200000, 2, 21, init_blocks=150),
    "propositions-wide-marks": lambda: gen.random_lts(40000, 160000, 40, 22, init_blocks=100),
    "product": lambda: permuted(gen.sync_product(4, 14, seed=23), 24),
}


@pytest.mark.parametrize("case", sorted(MANY_LARGE))
def test_rounds_reuse_tracked_entries(B, case):
    """The entries of tracked labels turn over while their labels split; the
    lock-step engine gives the iteration count."""
    L = MANY_LARGE[case]()
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst, L.init)
    ref, _ = run(B, L, 2)
    got, _ = run(B, L, 3)
    with B.Batch([L]) as b:
        out, its, _ = b.run()
        batched = b.split(out.numpy())[0]
    for blk, n_it in [(x, i) for x, i, _ in got] + [(batched, its[0])]:
        assert (blk == ks).all() and n_it == ref[0][1]
    assert got[0][2] == nb


@pytest.mark.parametrize("seed", [1, 2])
def test_rounds_algorithm2(B, seed):
    check(B, gen.kripke_uniform(1000, 5000, seed=seed), algorithm=2, engines=(0,))
    check(B, gen.random_lts(700, 1500, 1, seed, init_blocks=3), algorithm=2, engines=(0,))


@pytest.mark.parametrize("lds", [0, 2000, 30000, 70000])
def test_batch_rounds_default_workgroup(B, lds):
    """The batched kernel at its default workgroup size, from the whole LDS
    down to a budget that holds neither the table nor the label bitmaps."""
    insts = [CASES[c]() for c in ("n1", "n64", "kripke", "wide-marks", "chain", "fan-out", "hub",
                                  "planted-2-actions", "no-transitions")]
    with B.Batch(insts) as b:
        b.set_option(B.BOPT_LDS_LIMIT, lds)
        b.set_option(B.BOPT_GRID, 4)  # a workgroup takes several instances
        out, its, st = b.run()
        blocks = b.split(out.numpy())
    assert st["workgroup_size"] == 1024
    for k, L in enumerate(insts):
        ref = oracle.alg3_trace(L.n, L.K, L.src, L.lab, L.dst, L.init)
        assert (blocks[k] == ref["block"]).all() and its[k] == ref["iters"], (k, L.name)


@pytest.mark.parametrize("lds", [0, 1024, 1 << 14, 40000])
def test_mixed_batch_default_workgroup(B, lds):
    """Uneven instances, empty ones among them, at the default 1024 threads."""
    from test_gpu_batch import mixed_instances, check as check_batch
    insts = mixed_instances()
    with B.Batch(insts) as b:
        b.set_option(B.BOPT_LDS_LIMIT, lds)
        b.set_option(B.BOPT_GRID, 7)
        out, its, st = b.run()
        blocks = b.split(out.numpy())
    assert st["workgroup_size"] == 1024
    check_batch(B, insts, blocks, its)
