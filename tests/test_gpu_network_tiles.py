"""GPU: the network's matrix kernels at the edges of their tiles, and the
learned policy by one workgroup against the policy by kernels."""
from contextlib import closing

import numpy as np
import pytest

import oracle
from oracle import mlp as om
from paper_2105_11788_amd import gen

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2105_11788_amd import bisim
    bisim.load_library()
    assert bisim.device_count() > 0, "GPU tests need a GPU"
    return bisim


def inputs(rows, F, seed):
    rng = np.random.default_rng(seed)
    x = np.log1p(rng.poisson(rng.gamma(1.0, 4.0, (rows, F)))).astype(np.float32)
    t = np.log1p(rng.poisson(2.0, rows)).astype(np.float32)
    return om.he_init(F, seed), x, t


# a tile is 16 rows, a workgroup four tiles; 16,384 rows fill the training grid
@pytest.mark.parametrize("rows,F", [(1, 19), (15, 19), (16, 19), (17, 1), (63, 4), (65, 32),
                                    (1000, 19), (16385, 19), (70000, 20)])
def test_network_tile_edges(B, rows, F):
    w, x, t = inputs(rows, F, rows + F)
    y, c = om.forward(w, x, F)
    # a dot product of L terms (and a bias) errs by at most (L + 1) 2^-24 times
    # the sum of its absolute terms; the layers' errors pass through |W|
    u, p = 2.0 ** -24, {k: np.abs(v) for k, v in c["p"].items()}
    e1 = (F + 4) * u * (np.abs(c["x"]) @ p["W1"].T + p["b1"])
    e2 = e1 @ p["W2"].T + 66 * u * (c["h1"] @ p["W2"].T + p["b2"])
    ey = e2 @ p["w3"] + 68 * u * (c["h2"] @ p["w3"] + p["b3"][0])
    with closing(B.MLP(F, init=w)) as m:
        got = m.forward(x)
        assert (np.abs(got - y) <= 2 * ey).all()
        bits = (om.bf16_round(x).view(np.uint32) >> 16).astype(np.uint16)
        assert (m.forward_bf16(bits) == got).all()
        loss, grad = m.train_step(x, t, 0.0, want_grad=True)
        ref_loss, ref = om.loss_and_grad(w, x, t, F)
        assert abs(loss - ref_loss) <= 1e-5 * abs(ref_loss)
        # a unit whose pre-activation rounds to the other side of zero moves a
        # gradient by one row's share; else the fp32 sums are exact to 1e-5
        assert np.abs(grad - ref).max() <= 1e-3 * np.abs(ref).max()


LEARNED = {
    "n1": lambda: gen.random_lts(1, 2, 1, 1),
    "n64": lambda: gen.random_lts(64, 250, 3, 2),
    "n65": lambda: gen.random_lts(65, 300, 70, 3),
    "kripke": lambda: gen.kripke_uniform(700, 3500, seed=4),
    # more than 64 actions per state: the mark words stay in global memory
    "wide": lambda: gen.LTS(120, 200, np.repeat(np.arange(120), 90),
                            np.random.default_rng(3).integers(0, 200, 120 * 90),
                            np.random.default_rng(4).integers(0, 120, 120 * 90)),
    "n2048": lambda: gen.uniform_lts(2048, 5.0, 6, 5),
    "n2049": lambda: gen.uniform_lts(2049, 5.0, 6, 6),  # four kernels again
}


@pytest.mark.parametrize("case", sorted(LEARNED))
def test_learned_by_one_workgroup(B, case):
    L = LEARNED[case]()
    ks, nb = oracle.ks_coarsest(L.n, L.K, L.src, L.lab, L.dst, L.init)
    mlp = B.MLP(init=om.he_init(19, 11))
    t = lambda a: None if a is None else B.DeviceArray.from_numpy(a, np.int32)
    res = []
    for engine in (0, 2):
        with B.LTS(t(L.src), t(L.lab), t(L.dst), L.n, L.K, t(L.init)) as h:
            h.set_option(B.OPT_ENGINE, engine)
            B.set_splitter_policy(h, B.POLICY_LEARNED, mlp, 16)
            tr = h.set_trace(3 * L.n + 2)
            blk, st = h.run()
            assert (blk.numpy() == ks).all() and st.blocks == nb
            res.append((st.iterations, tr[0].numpy()[:st.iterations].tolist(),
                        tr[1].numpy()[:st.iterations].tolist()))
            if engine == 0:
                assert h.run_config() == ((1, 1) if L.n <= 2048 else h.run_config())
    mlp.close()
    assert res[0] == res[1]
