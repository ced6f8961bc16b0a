"""A handle's device memory: pieces given back make room again (on the CPU),
and runs on one handle take no more memory than the first ones did (GPU)."""
import ctypes
import itertools
import os
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2105_11788_amd", "csrc")
P = ctypes.c_void_p

PIECES = r"""
#include <stdint.h>
#include "pieces.h"
using bisim::Pieces;
extern "C" {
Pieces* make(size_t capacity) { return new Pieces(capacity); }
void drop(Pieces* p) { delete p; }
int64_t cut(Pieces* p, size_t bytes) { size_t at; return p->cut(bytes, &at) ? (int64_t)at : -1; }
void give_back(Pieces* p, size_t at) { p->give_back(at); }
size_t used(Pieces* p) { return p->used(); }
}
"""


@pytest.fixture(scope="module")
def pieces(tmp_path_factory):
    d = tmp_path_factory.mktemp("pieces")
    (d / "pieces.cpp").write_text(PIECES)
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-fPIC", "-shared", "-Wall", "-I", CSRC,
                           str(d / "pieces.cpp"), "-o", str(d / "pieces.so")])
    lib = ctypes.CDLL(str(d / "pieces.so"))
    lib.make.restype, lib.cut.restype, lib.used.restype = P, ctypes.c_int64, ctypes.c_size_t
    lib.make.argtypes, lib.drop.argtypes, lib.used.argtypes = [ctypes.c_size_t], [P], [P]
    lib.cut.argtypes = lib.give_back.argtypes = [P, ctypes.c_size_t]
    return lib


@pytest.mark.parametrize("order", list(itertools.permutations(range(4))))
def test_pieces_given_back_in_any_order(pieces, order):
    p = pieces.make(1000)
    stays = pieces.cut(p, 100)
    for _ in range(2):
        at = [pieces.cut(p, b) for b in (10, 200, 30, 256)]
        assert at == [100, 110, 310, 340]
        assert pieces.cut(p, 405) == -1 and pieces.used(p) == 596
        for i in order:
            pieces.give_back(p, at[i])
        assert pieces.used(p) == 100
    assert pieces.cut(p, 900) == 100 and pieces.cut(p, 1) == -1
    pieces.give_back(p, stays)  # below a piece in use: no room yet
    assert pieces.used(p) == 1000
    pieces.drop(p)


def pool_bytes(B):
    """bytes in use of the device's default memory pool"""
    H = B.hip()
    pool, used = P(), ctypes.c_uint64(0)
    assert H.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert H.hipDeviceSynchronize() == 0
    assert H.hipMemPoolGetAttribute(pool, 0x7, ctypes.byref(used)) == 0  # used, now
    return used.value


@pytest.mark.gpu
def test_runs_on_a_handle_take_no_more_memory():
    """Runs scan arrays of 5M states, and the signature rounds sort them:
    temporaries of 10 KB, of which 1 MiB would be a new chunk."""
    from paper_2105_11788_amd import bisim as B
    n = 5_000_000
    one = B.DeviceArray.from_numpy(np.zeros(1, np.int32), np.int32)
    out = B.DeviceArray(n, np.int32)
    with B.LTS(one, one, one, n, 1, None) as h:
        h.set_option(B.OPT_ENGINE, 3)
        algorithms = (100, 3)
        for a in algorithms:
            h.set_option(B.OPT_ALGORITHM, a)
            h.run(out)
        before = pool_bytes(B)
        for a, runs in zip(algorithms, (100, 300)):
            h.set_option(B.OPT_ALGORITHM, a)
            for _ in range(runs):
                _, st = h.run(out)
            assert st.blocks == 2  # the state with a transition, the others
            print(f"algorithm {a}: {pool_bytes(B) - before} bytes more", flush=True)
        assert pool_bytes(B) == before


@pytest.mark.gpu
@pytest.mark.parametrize("actions", [3, 70, 200])
def test_load_leaves_no_temporaries(actions):
    """With at most 64 actions, and with more: states of up to 64 and (200)
    of more than 64 of them.  The bound is what stays: 24 bytes per state and
    8 to 9 per transition of the load, 150 per state of the run, 8 per
    transition of its layout by source; 2 MiB for rounding."""
    from paper_2105_11788_amd import bisim as B, gen
    L = (gen.uniform_lts(200_000, 100.0, actions, 1) if actions == 200
         else gen.uniform_lts(300_000, 6.0, actions, 1))
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    before = pool_bytes(B)
    with B.LTS(*dev, L.n, L.K, None) as h:
        h.set_option(B.OPT_ENGINE, 3)
        h.set_option(B.OPT_ITER_LIMIT, 2)
        with pytest.raises(B.BisimError):
            h.run()
        extra = 16 * L.m // 64 if actions == 200 else 0  # mark words beyond one per state
        assert pool_bytes(B) - before <= 174 * L.n + 17 * L.m + extra + (2 << 20)
    assert pool_bytes(B) == before


@pytest.mark.gpu
def test_runs_within_less_memory(monkeypatch, tmp_path):
    """What fits is run: without the layout that tracks large splitters, and
    without the member lists (by the engine that needs none), down to what
    loading takes.  Loads may fail, automatic runs never do."""
    from paper_2105_11788_amd import bisim as B, gen
    import oracle
    monkeypatch.setenv("BISIM_TUNE_CACHE", str(tmp_path / "tune.txt"))
    L = gen.planted_quotient(1500, 4.0, 3, seed=5)
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst)
    dev = [B.DeviceArray.from_numpy(a, np.int32) for a in (L.src, L.lab, L.dst)]
    seen, its = [], set()
    for limit in range(1 << 20, 12 << 20, 1 << 18):
        monkeypatch.setenv("BISIM_HANDLE_LIMIT", str(limit))
        try:
            h = B.LTS(*dev, L.n, L.K, None)
        except B.BisimError as e:
            assert e.status == B.E_NOMEM and not seen
            continue
        with h:
            for _ in range(2):
                out, st = h.run()
                assert (out.numpy() == ks).all() and st.blocks == nb
                its.add(st.iterations)
            seen.append(h.run_config()[0])
            h.set_option(B.OPT_ENGINE, 3)
            if seen[-1] == 3:
                h.run()
            else:
                with pytest.raises(B.BisimError) as e:
                    h.run()
                assert e.value.status == B.E_NOMEM
                h.set_option(B.OPT_ENGINE, 0)  # the handle stays usable
                assert (h.run()[0].numpy() == ks).all()
    assert len(its) == 1 and seen == sorted(seen) and {2, 3} <= set(seen)


@pytest.mark.gpu
def test_batch_within_less_memory(monkeypatch):
    from paper_2105_11788_amd import bisim as B, gen
    import oracle
    insts = [gen.planted_quotient(300, 30.0, 3, seed=s) for s in (1, 2)]
    refs = [oracle.alg3_trace(L.n, L.K, L.src, L.lab, L.dst) for L in insts]
    ran = failed = 0
    for limit in range(1 << 20, 12 << 20, 1 << 18):
        monkeypatch.setenv("BISIM_HANDLE_LIMIT", str(limit))
        try:
            b = B.Batch(insts)
        except B.BisimError as e:
            assert e.status == B.E_NOMEM and not ran
            failed += 1
            continue
        with b:
            b.set_option(B.BOPT_GRID, 2)
            out, its, _ = b.run()
            for x, n_it, r in zip(b.split(out.numpy()), its, refs):
                assert (x == r["block"]).all() and n_it == r["iters"]
            ran += 1
    # what a load takes and leaves, a chunk and a step of the limit for rounding;
    # the layout by source would be 8 bytes per transition more
    n, m = sum(L.n for L in insts), sum(L.m for L in insts)
    print(f"n {n} m {m}: loads from {(1 << 20) + failed * (1 << 18)} on", flush=True)
    assert ran and 8 * m > 2 << 20
    assert (1 << 20) + failed * (1 << 18) <= 8 * m + 88 * n + (1 << 20) + (1 << 18)
