"""The calls that this library is used for, over the sizes they are used at.

Each case is one user-level call: an LTS whose transition arrays are on the
device is loaded, refined and its block ids read back (the single-instance
form, the signature baseline, the learned splitter), a loaded batch is refined,
or the splitter network is trained or evaluated.  Sizes follow the workloads of
the benchmark and the tests: the Kripke structure of 1000 states, Fan_out_n,
the labelled chain, the chain-sized LTS with as many actions as transitions,
the synchronised product, the planted quotient of a million states and the
uneven batch.  Inputs are drawn from the seed alone.
"""
import math

import numpy as np
import torch

from paper_2105_11788_amd import bisim, gen

FEATURES = bisim.POLICY_FEATURES
HIDDEN = 64


def listed():
    return [
        # the smallest useful LTS (one component of a model): launch latency
        dict(name="random-100", kind="random", n=100, degree=4.0, actions=4, props=0, alg=3),
        # a Kripke structure with one proposition, the paper's smallest setting
        dict(name="kripke-1k", kind="random", n=1000, degree=5.0, actions=1, props=2, alg=3),
        # a mid-sized unstructured state space: tens of thousands of iterations
        dict(name="uniform-20k", kind="random", n=20000, degree=6.0, actions=8, props=0, alg=3),
        # the paper's Fan_out family: two hubs and a chain, one large splitter
        dict(name="fan-out-2000", kind="fan_out", n=2000),
        # two copies of a deep chain: the worst case of the iteration count
        dict(name="chains-8k", kind="chain", n=8000),
        # about as many actions as transitions (a row of the paper's table):
        # the one-pass preprocessing, then one iteration per block
        dict(name="many-actions-25k", kind="random", n=25217, degree=1.0, actions=25216, props=0,
             alg=3),
        # a synchronised product of four processes: structured, no symmetry left
        dict(name="product-20k", kind="product", procs=4, length=12),
        # a large LTS with much symmetry, the benchmark's default workload
        dict(name="planted-1M", kind="planted", q=50000, degree=8.0, actions=16, alg=3),
        # the multi-way signature rounds on a large LTS
        dict(name="signature-2M", kind="planted", q=100000, degree=8.0, actions=16, alg=100),
        # many independent LTSs of uneven size in one launch
        dict(name="batch-256", kind="batch", count=256, n_hi=40000),
        # a training-sized LTS refined with the network choosing the splitter
        dict(name="learned-1k", kind="learned", n=1000, actions=1),
        # one training step of the splitter network on the rows of a collection
        dict(name="mlp-train-32k", kind="mlp", rows=32768, op="train"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["random", "random", "fan_out", "chain", "many", "product", "planted",
                       "planted", "signature", "batch", "batch", "learned", "mlp"])
    if kind == "random":
        K = rng.choice([1, 1, 2, 3, 8, 20, 64])
        alg = rng.choice([2, 3]) if K == 1 else 3
        return dict(kind="random", n=_log(rng, 100, 20000), degree=round(rng.uniform(1.5, 8.0), 1),
                    actions=K, props=2 if alg == 2 else rng.choice([0, 2, 3]), alg=alg)
    if kind == "many":
        n = _log(rng, 1000, 25000)
        return dict(kind="random", n=n, degree=1.0, actions=n - 1, props=0, alg=3)
    if kind == "fan_out":
        return dict(kind="fan_out", n=_log(rng, 50, 2200))
    if kind == "chain":
        return dict(kind="chain", n=2 * _log(rng, 150, 4500))
    if kind == "product":
        procs = rng.choice([3, 4])
        return dict(kind="product", procs=procs,
                    length=rng.randint(8, 27) if procs == 3 else rng.randint(5, 12))
    if kind == "planted":
        return dict(kind="planted", q=_log(rng, 300, 40000), degree=round(rng.uniform(4, 10), 1),
                    actions=rng.choice([2, 5, 16, 40]), alg=3)
    if kind == "signature":
        return dict(kind="planted", q=_log(rng, 2000, 90000), degree=round(rng.uniform(4, 10), 1),
                    actions=rng.choice([5, 16, 40]), alg=rng.choice([100, 101]))
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(64, 256), n_hi=_log(rng, 1500, 30000))
    if kind == "learned":
        return dict(kind="learned", n=_log(rng, 200, 1000), actions=rng.choice([1, 64]))
    return dict(kind="mlp", rows=_log(rng, 500, 32000), op=rng.choice(["train", "forward", "bf16"]))


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _planted(q, degree, K, seed):
    """gen.planted_quotient's construction on the GPU (a quotient graph with
    Zipf labels, 1..40 copies per node, permuted ids, shuffled edges); the
    copies are a shuffled even spread, so that n is the same for every seed."""
    d = torch.device("cuda")
    g = torch.Generator(device=d).manual_seed(seed)
    rand = lambda hi, size: torch.randint(0, hi, (size,), generator=g, device=d)
    deg = torch.poisson(torch.full((q,), float(degree), device=d), generator=g).long()
    src = torch.repeat_interleave(torch.arange(q, device=d), deg)
    p = torch.arange(1, K + 1, device=d, dtype=torch.float64) ** -1.1
    cdf = torch.cumsum(p / p.sum(), 0)
    u = torch.rand(src.numel(), generator=g, device=d, dtype=torch.float64)
    lab = torch.searchsorted(cdf, u).clamp_(max=K - 1)
    key = torch.unique((src * K + lab) * q + rand(q, src.numel()))
    qdst, lab, src = key % q, key // q % K, key // (q * K)
    c = (torch.arange(q, device=d) % 40 + 1)[torch.randperm(q, generator=g, device=d)]
    end = torch.cumsum(c, 0)
    start, n = end - c, int(end[-1])
    reps = c[src]
    e = torch.repeat_interleave(torch.arange(src.numel(), device=d), reps)
    first = torch.cumsum(reps, 0) - reps
    tgt = qdst[e]
    u_pos = start[src[e]] + torch.arange(e.numel(), device=d) - first[e]
    r = torch.rand(e.numel(), generator=g, device=d, dtype=torch.float64)
    v_pos = start[tgt] + (r * c[tgt]).long()
    perm = torch.randperm(n, generator=g, device=d)
    order = torch.randperm(e.numel(), generator=g, device=d)
    host = lambda t: t[order].int().cpu().numpy()
    return gen.LTS(n, K, host(perm[u_pos]), host(lab[e]), host(perm[v_pos]))


def _permuted(L, rng):
    """The same LTS under another numbering of its states."""
    p = rng.permutation(L.n)
    order = rng.permutation(L.m)
    return gen.LTS(L.n, L.K, p[L.src[order]], L.lab[order], p[L.dst[order]])


def _lts(case, seed):
    rng = np.random.default_rng(seed)
    kind = case["kind"]
    if kind == "fan_out":
        return _permuted(gen.fan_out(case["n"]), rng)
    if kind == "chain":
        one = gen.chain_tail(case["n"] // 2)
        two = lambda a, shift: np.concatenate([a, a + shift])
        return _permuted(gen.LTS(2 * one.n, 2, two(one.src, one.n), two(one.lab, 0),
                                 two(one.dst, one.n)), rng)
    if kind == "product":
        return _permuted(gen.sync_product(case["procs"], case["length"], seed=seed), rng)
    if kind == "planted":
        return _planted(case["q"], case["degree"], case["actions"], seed)
    if kind == "learned":
        n = case["n"]
        return (gen.kripke_uniform(n, 5 * n, seed) if case["actions"] == 1
                else gen.uniform_zipf(n, 5 * n, case["actions"], seed))
    n, m = case["n"], int(case["n"] * case["degree"])
    return gen.random_lts(n, m, case["actions"], seed, init_blocks=case["props"])


def _batch(case, seed):
    """An uneven batch: sizes spread evenly over the logarithm, in a shuffled
    order; planted quotients and uniform LTSs alternate, as gen.batch has them."""
    rng = np.random.default_rng(seed)
    count, insts = case["count"], []
    at = (np.arange(count) + 0.5) / count
    for k, n in enumerate((100 * (case["n_hi"] / 100) ** at).astype(int)):
        s, K = int(rng.integers(1 << 40)), 1 + k * 7 % 32
        insts.append(_planted(max(1, round(n / 20.5)), 6.0, K, s) if k % 2 == 0
                     else gen.uniform_lts(int(n), 6.0, K, s))
    order = np.random.default_rng(count).permutation(count)
    return [insts[k] for k in order]


def _weights(rng):
    """He-normal network parameters in the library's order, zero biases."""
    z = lambda k: np.zeros(k, np.float32)
    w = lambda rows, cols, s: rng.normal(0, s, rows * cols).astype(np.float32)
    return np.concatenate([w(HIDDEN, FEATURES, (2.0 / FEATURES) ** 0.5), z(HIDDEN),
                           w(HIDDEN, HIDDEN, (2.0 / HIDDEN) ** 0.5), z(HIDDEN),
                           w(1, HIDDEN, (1.0 / HIDDEN) ** 0.5), z(1)])


def _rows(case, seed):
    """Feature rows as a collection gives them: log1p of block size and
    transition counts, log1p of the age, the used flag; targets log1p(splits)."""
    rng = np.random.default_rng(seed)
    w = _weights(rng)
    B = case["rows"]
    x = np.empty((B, FEATURES), np.float32)
    x[:, 0] = np.log1p(rng.geometric(0.2, B))
    x[:, 1:17] = np.log1p(rng.poisson(rng.gamma(1.0, 4.0, (B, 16))))
    x[:, 17] = np.log1p(rng.integers(0, 1500, B))
    x[:, 18] = rng.integers(0, 2, B)
    t = np.log1p(rng.poisson(2.0, B)).astype(np.float32)
    return w, x, t


def _bf16(x):
    """float32 values rounded to bfloat16 (to nearest, ties to even)."""
    return torch.from_numpy(np.ascontiguousarray(x, np.float32)).to(torch.bfloat16)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mlp":
        w, x, t = _rows(case, seed)
        x = (bisim.DeviceArray.from_numpy(_bf16(x).view(torch.int16).numpy().view(np.uint16))
             if case["op"] == "bf16" else bisim.DeviceArray.from_numpy(x))
        return dict(kind=kind, op=case["op"], mlp=bisim.MLP(FEATURES, init=w), x=x,
                    t=bisim.DeviceArray.from_numpy(t))
    if kind == "batch":
        b = bisim.Batch(_batch(case, seed))
        return dict(kind=kind, batch=b, out=bisim.DeviceArray(b.N))
    L = _lts(case, seed)
    up = lambda a: None if a is None else bisim.DeviceArray.from_numpy(a, np.int32)
    s = dict(kind=kind, n=L.n, K=L.K, src=up(L.src), lab=up(L.lab), dst=up(L.dst),
             init=up(L.init), alg=case.get("alg", 3))
    if kind == "learned":
        s["mlp"] = bisim.MLP(FEATURES, init=_weights(np.random.default_rng(seed)))
    return s


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
def run(s):
    if s["kind"] == "mlp":
        if s["op"] == "train":
            loss, grad = s["mlp"].train_step(s["x"], s["t"], 3e-3, want_grad=True)
            return dict(loss=loss, grad=grad)
        f = s["mlp"].forward if s["op"] == "forward" else s["mlp"].forward_bf16
        return dict(y=f(s["x"]))
    if s["kind"] == "batch":
        out, its, _ = s["batch"].run(s["out"])
        return dict(blocks=out.numpy(), iterations=its)
    with bisim.LTS(s["src"], s["lab"], s["dst"], s["n"], s["K"], s["init"]) as h:
        if s["alg"] != 3:
            h.set_option(bisim.OPT_ALGORITHM, s["alg"])
        if "mlp" in s:
            bisim.set_splitter_policy(h, bisim.POLICY_LEARNED, s["mlp"])
        out, st = h.run()
        return dict(blocks=out.numpy(), iterations=st.iterations, count=st.blocks)


# --------------------------------------------------------------------------
# what a pass cannot do without, and the network's values in 64 bits
# --------------------------------------------------------------------------
def work(case):
    """Transitions (three ids each) and the initial partition read once, block
    ids written once; for the network its rows and its multiply-adds."""
    kind = case["kind"]
    if kind == "mlp":
        macs = FEATURES * HIDDEN + HIDDEN * HIDDEN + HIDDEN
        B, train = case["rows"], case["op"] == "train"
        row = FEATURES * (2 if case["op"] == "bf16" else 4) + 4
        return dict(bytes=B * row + 4 * (macs + 2 * HIDDEN + 1), flops=2 * B * macs * (3 if train else 1))
    if kind == "batch":
        n = case["count"] * (case["n_hi"] - 100) / math.log(case["n_hi"] / 100)
        m = 6.0 * n
    elif kind == "planted":
        n = 20.5 * case["q"]
        m = n * case["degree"]
    elif kind == "product":
        n = case["length"] ** case["procs"]
        m = n * case["procs"]
    elif kind == "fan_out":
        n, m = case["n"], 3 * case["n"] - 3
    elif kind == "chain":
        n, m = case["n"], case["n"] - 2
    else:
        n = case["n"]
        m = n * case.get("degree", 5.0)
    init = 4 * n if case.get("props") or (kind == "learned" and case["actions"] == 1) else 0
    return dict(bytes=12 * m + 4 * n + init, flops=0)


def exact(case, seed):
    """Partitions and iteration counts are whole numbers; the network's outputs
    from its definition (parameters and inputs rounded to bfloat16) in 64 bits."""
    if case["kind"] != "mlp":
        return None
    w, x, t = _rows(case, seed)
    p = _bf16(w).double()
    x, t = _bf16(x).double(), torch.from_numpy(t).double()
    H, F = HIDDEN, FEATURES
    W1, b1, W2, b2, w3, b3 = torch.split(p, [H * F, H, H * H, H, H, 1])
    W1, W2 = W1.view(H, F), W2.view(H, H)
    z1 = x @ W1.T + b1
    h1 = z1.clamp(min=0)
    z2 = h1 @ W2.T + b2
    h2 = z2.clamp(min=0)
    y = h2 @ w3 + b3
    if case["op"] != "train":
        return dict(y=y)
    dy = 2.0 * (y - t) / y.numel()
    d2 = torch.outer(dy, w3) * (z2 > 0)
    d1 = (d2 @ W2) * (z1 > 0)
    grad = torch.cat([(d1.T @ x).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0),
                      h2.T @ dy, dy.sum().view(1)])
    return dict(loss=float(((y - t) ** 2).mean()), grad=grad)
