"""The rounds of one workgroup (rounds_dev.h), compiled for the host and run
lane by lane against the lock-step oracle.  Constants are lowered so that the
borders they draw lie within small LTSs; whole numbers, no tolerance."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2105_11788_amd import gen

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2105_11788_amd", "csrc")
P = ctypes.c_void_p


class Run(ctypes.Structure):
    _fields_ = [("n", ctypes.c_int32), ("m", ctypes.c_int32), ("K", ctypes.c_int32),
                ("start", P), ("in_ptr", P), ("in_src", P), ("in_ord", P),
                ("out_ptr", P), ("out_dst", P), ("out_ord", P),
                ("rcpp", ctypes.c_int32), ("lds_bytes", ctypes.c_int32),
                ("bitmaps_in_lds", ctypes.c_int32), ("either", ctypes.c_int32),
                ("seed", ctypes.c_uint32), ("block", P), ("iterations", P)]


def compiled(folder, constants, header="rounds_dev.h", model="rounds_model.cpp"):
    """The model with some of the header's constants replaced."""
    text = open(os.path.join(CSRC, header)).read()
    for name, (was, now) in constants.items():
        assert text.count(f"{name} = {was}") == 1, name
        text = text.replace(f"{name} = {was}", f"{name} = {now}")
    open(os.path.join(folder, header), "w").write(text)
    for f in ("internal.h", model):
        shutil.copy(os.path.join(HERE, "host_model", f), folder)
    so = os.path.join(folder, "model.so")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-w",
                           "-I", str(folder), os.path.join(folder, model), "-o", so])
    return ctypes.CDLL(so)


def run(lib, L, lds=60000, either=False, track=True, bitmaps=True, seed=1):
    pre = oracle.preprocess(L.n, L.K, L.src, L.lab, L.dst, L.init)

    def grouped(by, other):
        order = np.argsort(pre[by], kind="stable")
        ptr = np.searchsorted(pre[by][order], np.arange(L.n + 1)).astype(np.uint32)
        return [ptr] + [np.ascontiguousarray(pre[x][order]) for x in (other, "order")]

    arrays = ([pre["pre_block"].copy()] + grouped("s_dst", "s_src") + grouped("s_src", "s_dst"))
    block, its = np.empty(L.n, np.int32), np.zeros(1, np.int64)
    p = [a.ctypes.data_as(P) for a in arrays]
    if not track:
        p[4:] = [None] * 3
    r = Run(L.n, L.m, L.K, *p, 0, lds, bitmaps, either, seed,
            block.ctypes.data_as(P), its.ctypes.data_as(P))
    assert lib.model_run(ctypes.byref(r)) == 0
    return block, int(its[0])


def check(lib, L, **options):
    ref = oracle.alg3_trace(L.n, L.K, L.src, L.lab, L.dst, L.init)
    block, its = run(lib, L, **options)
    assert (block == ref["block"]).all() and its == ref["iters"], (L.name, options, its,
                                                                   ref["iters"])


@pytest.fixture(scope="module")
def few_entries(tmp_path_factory):
    """As many tracked labels as candidates, tracked from the first round and
    from few transitions on, so that entries turn over all the time."""
    return compiled(tmp_path_factory.mktemp("few"), {
        "kCand": ("32", "8"), "kTracked": ("64", "8"), "kTrackEdges": ("384", "3"),
        "kTrackEdgesDense": ("1536", "3"), "kTrackAfter": ("8", "0")})


# schedules of the lanes under which the splitter's lost states were written
# into the label that had been given its entry (other iteration counts)
@pytest.mark.parametrize("either,lds,seed", [
    (True, 29000, 759097991), (True, 29000, 801935232), (True, 29000, 718905886),
    (True, 33000, 422976252), (True, 33000, 220949275), (True, 33000, 848167431),
    (True, 60000, 669684967), (True, 60000, 373683345),
    (False, 29000, 320150180), (False, 60000, 758017750), (False, 60000, 21045789)])
def test_tracked_entry_of_the_splitter_is_taken(few_entries, either, lds, seed):
    """A stable label can be given the entry of the splitter of the same round."""
    check(few_entries, gen.sync_product(3, 8, seed=826946041), lds=lds, either=either, seed=seed)


@pytest.fixture(scope="module")
def short_keys(tmp_path_factory):
    """Table keys with 6 bits for the state: 63 states at most have them."""
    return compiled(tmp_path_factory.mktemp("keys"), {"kKeyBits": ("27", "6")})


@pytest.mark.parametrize("track", [False, True])
@pytest.mark.parametrize("n", [62, 63, 64, 65, 200])
def test_more_states_than_table_keys(short_keys, n, track):
    """A batch takes instances of more states than a table key has bits for."""
    for seed in range(3):
        L = gen.random_lts(n, 3 * n, 2, seed, init_blocks=3)
        check(short_keys, L, either=True, track=track, seed=seed)


@pytest.fixture(scope="module")
def grouped(tmp_path_factory):
    return compiled(tmp_path_factory.mktemp("grouped"), {}, "grouped_dev.h", "grouped_model.cpp")


# in-degrees: none at all, one state, hubs of several runs of transitions first
# and last, states without any before, between and after, runs that just fit
GROUPS = {
    "none": [0, 0, 0], "one": [1], "hub": [3000], "hub-first": [2000, 1, 1], "hub-last": [1, 0, 1500],
    "sparse": [0] * 400 + [1] + [0] * 300 + [2, 0, 1] + [0] * 500, "even": [1] * 1024,
    "run": [512, 0, 512, 1], "mixed": [k * 37 % 11 * (k % 3) for k in range(700)] + [900, 0, 0, 5],
}


@pytest.mark.parametrize("waves", [1, 3])
@pytest.mark.parametrize("case", sorted(GROUPS))
def test_each_in_transition_once(grouped, case, waves):
    degree = np.array(GROUPS[case], np.uint32)
    ptr = np.concatenate([[0], np.cumsum(degree)]).astype(np.uint32)
    m = int(ptr[-1])
    target, visits = np.full(max(m, 1), 77, np.uint32), np.zeros(max(m, 1), np.uint32)
    grouped.visit(len(degree), ptr.ctypes.data_as(P), waves, target.ctypes.data_as(P),
                  visits.ctypes.data_as(P))
    assert (visits[:m] == 1).all() and visits[m:].sum() == 0
    assert (target[:m] == np.repeat(np.arange(len(degree)), degree)).all()


@pytest.fixture(scope="module")
def shipped(tmp_path_factory):
    return compiled(tmp_path_factory.mktemp("shipped"), {})


def backward_chain(n):
    return gen.LTS(n, 1, np.arange(1, n), np.zeros(n - 1, int), np.arange(n - 1))


# blocks that lose more states than the tables of a split hold (128 here): all
# but the leader, interleaved halves, several blocks at once
LARGE = {
    "backward-chain": lambda: backward_chain(420),
    "backward-chain-permuted": lambda: gen.LTS(400, 1, *(
        (lambda p, L: (p[L.src], L.lab, p[L.dst]))(np.random.default_rng(3).permutation(400),
                                                    backward_chain(400)))),
    "fat": lambda: gen.planted_quotient(6, 3.0, 2, seed=4, copies_hi=300),
    "two-chains": lambda: gen.LTS(600, 2, np.arange(2, 600), np.zeros(598, int),
                                  np.arange(598), np.arange(600) % 2),
    "wide-marks": lambda: gen.random_lts(500, 700, 50, 5, init_blocks=2),
    "halves": lambda: gen.LTS(602, 3, np.concatenate([np.arange(600), np.arange(600), [600, 601]]),
                              np.concatenate([np.zeros(1200, int), [1, 2]]),
                              np.concatenate([600 + np.arange(600) % 2, np.arange(600) // 2,
                                              [600, 601]])),
}


# (the third budget holds neither the table nor the tables of a split)
@pytest.mark.parametrize("lds,bitmaps,either", [(60000, True, False), (24000, True, True),
                                                (3000, False, True)])
@pytest.mark.parametrize("case", sorted(LARGE))
def test_large_splits(shipped, case, lds, bitmaps, either):
    check(shipped, LARGE[case](), lds=lds, bitmaps=bitmaps, either=either, seed=lds)
