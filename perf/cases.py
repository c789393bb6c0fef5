"""The work measured on this framework: batches of flip-graph walks of every kind that
it runs, the steps around them (initialisation, population synchronisation, Resize, Brent
verification, invariants, lifting) and the proposal network (scoring, training, use).

Sizes are those of the repository's workloads (bench.py, learn.py, explore.py) or cut from
them so that a pass stays well below a second; draw() spreads them over the same ranges.
Every case is one call sequence of the public binding, as a program that uses it makes it.
"""
import math

import numpy as np
import torch

from paper_2511_20317_amd import tsf

# the four formats that one mixed batch holds
MIXED = "3,3,4 3,4,5 4,4,4 4,4,5"


def listed():
    return [
        # the smallest search: every launch and every dependent step of an iteration shows
        {"name": "walk_222_small", "kind": "walk", "formats": "2,2,2", "walks": 256,
         "iters": 1000, "warm": 0, "target": 7, "mode": 0, "objective": 0, "p_expand": 0.0},
        # the headline search, a batch that fills the chip
        {"name": "walk_333", "kind": "walk", "formats": "3,3,3", "walks": 65536,
         "iters": 10000, "warm": 2000, "target": 23, "mode": 0, "objective": 0, "p_expand": 0.0},
        # several formats in one launch, ranks up to 80
        {"name": "walk_mixed", "kind": "walk", "formats": MIXED, "walks": 65536,
         "iters": 1000, "warm": 1000, "target": 0, "mode": 0, "objective": 0, "p_expand": 0.0},
        # Z2 coefficients, an odd batch far smaller than the chip, with expands
        {"name": "walk_345_z2", "kind": "walk", "formats": "3,4,5", "walks": 1777,
         "iters": 2000, "warm": 1000, "target": 0, "mode": 1, "objective": 0, "p_expand": 0.01},
        # a large format: 64-bit factors, 378 terms
        {"name": "walk_679", "kind": "walk", "formats": "6,7,9", "walks": 8192,
         "iters": 1000, "warm": 300, "target": 0, "mode": 0, "objective": 0, "p_expand": 0.0},
        # the complexity-minimisation mode on schemes of a rank search
        {"name": "walk_333_additions", "kind": "walk", "formats": "3,3,3", "walks": 16384,
         "iters": 5000, "warm": 20000, "target": 0, "mode": 0, "objective": 1, "p_expand": 0.0},
        # one round of the exploratory search: walk, synchronise the population, resize
        {"name": "explore_round", "kind": "explore", "walks": 16384, "iters": 500,
         "capacity": 128, "rounds": 4, "mode": 0},
        # what follows every round of a search: the Brent check of every best scheme, and the
        # isotropy invariants of the schemes that are kept
        {"name": "check_best", "kind": "check", "formats": MIXED, "walks": 65536,
         "warm": 500, "mode": 0},
        # scoring the candidate flips of 4,096 walks
        {"name": "net_score", "kind": "score", "rows": 32768},
        # one training step of the proposal network at its training batch
        {"name": "net_train", "kind": "train", "rows": 4096},
        # walks with the learned proposal, as many iterations as its driver makes in a call
        {"name": "walk_learned", "kind": "learned", "formats": "3,3,3", "walks": 4096,
         "iters": 20, "warm": 1000},
        # signs for a Z2 scheme, by search
        {"name": "lift_223", "kind": "lift", "formats": "2,2,3", "walks": 1024, "iters": 4000,
         "max_nodes": 256, "max_subtrees": 16384},
    ]


# formats of the repository's workloads, by the size of their standard scheme
SMALL = ["2,2,2", "2,2,3", "2,3,3", "2,3,4", "3,3,3", "3,3,4", "2,5,5", "3,4,4", "3,3,5"]
MIDDLE = ["3,4,5", "4,4,4", "4,4,5", "3,5,5", "4,5,5"]
LARGE = ["4,5,12", "5,6,10", "6,7,9", "5,5,5"]


def _spread(rng, lo, hi):
    """an integer of [lo, hi], spread over its logarithm, odd and even alike"""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["walk"] * 5 + ["explore", "check", "score", "train", "learned", "lift"])
    if kind == "walk":
        size = rng.choice(["small", "small", "middle", "large"])
        if size == "small":
            walks, iters = _spread(rng, 64, 65536), _spread(rng, 500, 6000)
            formats = rng.choice(SMALL)
        elif size == "middle":
            walks, iters = _spread(rng, 64, 32768), _spread(rng, 200, 2000)
            formats = " ".join(rng.sample(MIDDLE, rng.choice([1, 1, 2, 3])))
        else:
            walks, iters = _spread(rng, 64, 6000), _spread(rng, 100, 800)
            formats = rng.choice(LARGE)
        return {"kind": "walk", "formats": formats, "walks": walks, "iters": iters,
                "warm": _spread(rng, 100, 800), "target": 0, "mode": rng.choice([0, 0, 0, 1]),
                "objective": rng.choice([0, 0, 0, 1]), "p_expand": rng.choice([0.0, 0.0, 0.01])}
    if kind == "explore":
        return {"kind": "explore", "walks": _spread(rng, 256, 16384),
                "iters": _spread(rng, 100, 500), "capacity": rng.choice([64, 96, 128]),
                "rounds": rng.randint(1, 5), "mode": rng.choice([0, 0, 1])}
    if kind == "check":
        if rng.random() < 0.3:
            return {"kind": "check", "formats": rng.choice(LARGE),
                    "walks": _spread(rng, 64, 2048), "warm": _spread(rng, 50, 300),
                    "mode": rng.choice([0, 0, 1])}
        return {"kind": "check", "formats": " ".join(rng.sample(SMALL + MIDDLE,
                                                                rng.randint(1, 4))),
                "walks": _spread(rng, 64, 65536), "warm": _spread(rng, 50, 1000),
                "mode": rng.choice([0, 0, 1])}
    if kind == "score":
        return {"kind": "score", "rows": _spread(rng, 100, 65536)}
    if kind == "train":
        return {"kind": "train", "rows": _spread(rng, 256, 16384)}
    if kind == "learned":
        return {"kind": "learned", "formats": rng.choice(["2,2,2", "3,3,3", "3,3,4"]),
                "walks": _spread(rng, 64, 4096), "iters": _spread(rng, 5, 40),
                "warm": _spread(rng, 100, 1000)}
    return {"kind": "lift", "formats": rng.choice(["2,2,2", "2,2,3", "2,2,4"]), "walks": 1024,
            "iters": _spread(rng, 1000, 4000), "max_nodes": _spread(rng, 16, 256),
            "max_subtrees": _spread(rng, 64, 16384)}


# ------------------------------------------------------------------------------------
# inputs
# ------------------------------------------------------------------------------------
def _formats(case):
    return [tuple(int(x) for x in f.split(",")) for f in case["formats"].split()]


def _groups(case, extra=8):
    fmts = _formats(case)
    share = case["walks"] // len(fmts)
    left = case["walks"] - share * len(fmts)
    return [(tsf.init_scheme(*f, mode=case.get("mode", 0)), share + (left if q == 0 else 0),
             f[0] * f[1] * f[2] + extra, case.get("target", 0)) for q, f in enumerate(fmts)]


def _params(case, seed, **kw):
    return tsf.walk_params(base_seed=int(seed) << 24, max_iters=10 ** 9, plateau=50000,
                           t_expand=int(round(case.get("p_expand", 0.0) * 2 ** 32)), **kw)


def _walked(ctx, case, seed, iters):
    """a batch from the standard schemes after `iters` iterations"""
    b = tsf.WalkBatch([g for g in _groups(case) if g[1] > 0], rec_cap=16)
    b.init(ctx)
    if iters:
        b.walk(ctx, _params(case, seed + 1), iters)
    return b


def _restart_from(b, ctx, which):
    """a batch whose start schemes are the current (0) or best (1) schemes of b"""
    n = b.n_walks
    out = tsf.WalkBatch.empty(n, b.capacity, b.mode, max_len=b.max_len, rec_cap=16)
    out.meta_from(b, which, np.zeros(n), np.zeros(n), np.zeros(n), r_cap_extra=8)
    return out


def _flip_records(rows, seed):
    """log records of `rows` applied flips (the 16 int64 words of a record), with factors of
    9 entries as (3,3,3) walks have them: one to four non-zero entries, ranks 23 to 27"""
    g = torch.Generator().manual_seed(int(seed) * 2 + 1)
    order = torch.rand((rows, 6, 9), generator=g).argsort(-1)
    count = 1 + (torch.rand((rows, 6, 1), generator=g) ** 2 * 4).long()
    nonzero = order < count
    negative = nonzero & (torch.rand((rows, 6, 9), generator=g) < 0.4)
    bit = 2 ** torch.arange(9)
    rank = 23 + (torch.rand(rows, generator=g) * 5).long()
    rec = torch.zeros((rows, 16), dtype=torch.int64)
    rec[:, 0] = torch.arange(rows)
    rec[:, 1] = rank | (rank << 32)
    rec[:, 2] = 5                                   # the slot of format (3,3,3)
    rec[:, 3:15:2] = (nonzero * bit).sum(-1)
    rec[:, 4:15:2] = (negative * bit).sum(-1)
    label = (torch.rand(rows, generator=g) < 0.25).float()
    sign = nonzero.double() - 2.0 * negative.double()
    return rec, label, sign, rank


def _features64(sign, rank):
    """the feature rows of _flip_records in 64 bits"""
    X = torch.zeros((sign.shape[0], 512), dtype=torch.float64)
    for q in range(6):
        X[:, 64 * q:64 * q + 9] = sign[:, q]
    X[:, 384 + 5] = 1.0
    X[torch.arange(sign.shape[0]), 400 + rank] = 1.0
    return X


def _weights(seed):
    rng = np.random.default_rng(int(seed))
    return [np.float32(w) for w in (
        rng.standard_normal((512, 256)) * np.sqrt(2 / 64), rng.standard_normal(256) * 0.1,
        rng.standard_normal((256, 256)) * np.sqrt(2 / 256), rng.standard_normal(256) * 0.1,
        rng.standard_normal(256) * np.sqrt(1 / 256), rng.standard_normal(1) * 0.1)]


def _moments(seed):
    """Adam's moments after some steps (a training run in progress)"""
    g = torch.Generator().manual_seed(int(seed) * 2)
    m = torch.randn(tsf.MLP_NPARAM, generator=g) * 3e-4
    v = (torch.rand(tsf.MLP_NPARAM, generator=g) * 0.9 + 0.1) * 1e-6
    m[-3:], v[-3:] = 0, 0                           # the padding behind b3
    return m, v


TRAIN_STEPS = 500        # steps that the measured one follows


def _network(seed, training=False):
    net = tsf.Mlp()
    net.set_params(*_weights(seed))
    if training:
        m, v = _moments(seed)
        net.adam_m.copy_(m)
        net.adam_v.copy_(v)
        net.step_count = TRAIN_STEPS
    return net


def prepare(case, seed):
    kind = case["kind"]
    ctx = tsf.Context()
    st = {"kind": kind, "case": case, "ctx": ctx}
    if kind == "walk":
        additions = case["objective"] == 1
        b = _walked(ctx, case, seed, case["warm"])
        if case["warm"]:
            b = _restart_from(b, ctx, 1 if additions else 0)
        if additions:                               # no target: the search never stops
            b.hdr.view(torch.int32).view(b.n_walks, tsf.HEADER_I32)[:, 5] = -10 ** 6
        st["batch"] = b
        st["prm"] = _params(case, seed, objective=case["objective"])
    elif kind == "explore":
        groups = [(tsf.init_scheme(*f, mode=case["mode"]), case["walks"] // 4,
                   f[0] * f[1] * f[2] + 8, 0)
                  for f in [(2, 2, 2), (2, 2, 3), (2, 3, 3), (3, 3, 3)]]
        a = tsf.WalkBatch(groups, capacity=case["capacity"], rec_cap=4)
        a.max_len = 64
        b = tsf.WalkBatch.empty(a.n_walks, a.capacity, a.mode, max_len=64, rec_cap=4)
        a.init(ctx)
        for q in range(case["rounds"]):             # the rounds before the measured one
            a.walk(ctx, _params(case, seed + 1 + q), 300)
            table, count = a.population_best()
            a.resize_into(b, table, count, int(seed), q)
            b.init(ctx)
            a, b = b, a
        st.update(batch=a, out=b, seed=int(seed), prm=_params(case, seed))
    elif kind == "check":
        st["batch"] = _walked(ctx, case, seed, case["warm"])
    elif kind == "score":
        rec = _flip_records(case["rows"], seed)[0].cuda()
        st["net"], st["X"] = _network(seed), tsf.features_from_log(rec)
    elif kind == "train":
        rec, label, _, _ = _flip_records(case["rows"], seed)
        st.update(net=_network(seed, True), rows=rec.cuda(), label=label.cuda())
    elif kind == "learned":
        st["batch"] = _restart_from(_walked(ctx, case, seed, case["warm"]), ctx, 0)
        st.update(prm=_params(case, seed), net=_network(seed),
                  ws=tsf.LearnWorkspace(case["walks"]))
    elif kind == "lift":
        b = _walked(ctx, dict(case, mode=1), seed, case["iters"])
        hdr = b.headers()
        low = np.flatnonzero(hdr["best_rank"] == hdr["best_rank"].min())
        st["scheme"] = b.scheme(int(low[int(seed) % low.size]), "best", hdr)
    return st


# ------------------------------------------------------------------------------------
# one pass
# ------------------------------------------------------------------------------------
def run(st):
    kind, case, ctx = st["kind"], st["case"], st["ctx"]
    if kind == "walk":
        b = st["batch"]
        b.init(ctx)
        b.walk(ctx, st["prm"], case["iters"])
        return b.hdr, b.cur, b.best, b.rec
    if kind == "explore":
        a, b = st["batch"], st["out"]
        a.init(ctx)
        a.walk(ctx, st["prm"], case["iters"])
        table, count = a.population_best()
        applied = a.resize_into(b, table, count, st["seed"], case["rounds"])
        b.init(ctx)
        return a.hdr, a.best, table, count, applied, b.hdr, b.start, b.cur
    if kind == "check":
        b = st["batch"]
        violated = b.verify_device(1)
        ranks, sums = b.invariants(1)
        return violated, ranks, sums
    if kind == "score":
        h1, h2, logit = st["net"].forward(st["X"])
        return h1.view(torch.bfloat16), h2.view(torch.bfloat16), logit
    if kind == "train":
        net, y = st["net"], st["label"]
        X = tsf.features_from_log(st["rows"])
        h1, h2, logit = net.forward(X)
        loss = net.backward(X, y, h1, h2, logit)
        net.step(lr=1e-3)
        return loss, net.grad, net.param, net.adam_m, net.adam_v, net.wbf.view(torch.bfloat16)
    if kind == "learned":
        b = st["batch"]
        b.init(ctx)
        b.walk_learned(ctx, st["prm"], st["net"], st["ws"], case["iters"])
        return b.hdr, b.cur, b.best
    info, scheme = tsf.lift(st["scheme"], max_nodes=case["max_nodes"],
                            max_subtrees=case["max_subtrees"])
    found = scheme.live() if scheme is not None else ()
    return info["status"], info["subtree"], info["subtrees"], found


# ------------------------------------------------------------------------------------
# what one pass cannot do without
# ------------------------------------------------------------------------------------
# 32-bit operations of a walk's iteration: the gate block and one attempt's block of the
# generator (100 each), and a flip on factors of one 32-bit word pair with its bookkeeping
ITER_OPS = 300
NET_FLOPS = 2 * (512 * 256 + 256 * 256 + 256)     # of a row, forward


def work(case):
    kind = case["kind"]
    if kind in ("walk", "explore", "check", "learned"):
        fmts = _formats(case) if "formats" in case else [(3, 3, 3)]
        ranks = sum(f[0] * f[1] * f[2] for f in fmts) / len(fmts)
        scheme = case["walks"] * ranks * 48.0
        header = case["walks"] * 176.0
    if kind == "walk":
        # starts in, current and best schemes out, headers in and out
        return {"bytes": 3 * scheme + 2 * header,
                "flops": float(ITER_OPS) * case["walks"] * case["iters"]}
    if kind == "explore":
        return {"bytes": 6 * scheme + 4 * header,
                "flops": float(ITER_OPS) * case["walks"] * case["iters"]}
    if kind == "check":
        return {"bytes": scheme + header + case["walks"] * (8 + 3 * ranks + 12),
                "flops": 10.0 * case["walks"] * ranks}
    if kind == "score":
        return {"bytes": case["rows"] * (1024.0 + 512 + 512 + 4) + 2 * 196864,
                "flops": float(case["rows"]) * NET_FLOPS}
    if kind == "train":
        # records and labels in; masters and moments in and out, gradients and copies out
        return {"bytes": case["rows"] * 132.0 + tsf.MLP_NPARAM * 28.0 + tsf.MLP_NBF16 * 2.0,
                "flops": float(case["rows"]) * (3 * NET_FLOPS - 2 * 512 * 256)}
    if kind == "learned":
        # per iteration the candidates of eight rows a walk are scored
        return {"bytes": 3 * scheme + 2 * header,
                "flops": 8.0 * case["walks"] * case["iters"] * NET_FLOPS}
    m, n, p = _formats(case)[0]
    return {"bytes": 4.0 * case["max_subtrees"],
            "flops": 2.0 * case["max_subtrees"] * (m * n * p) ** 2}


# ------------------------------------------------------------------------------------
# the network in 64 bits
# ------------------------------------------------------------------------------------
def _net64(w, X):
    W1, b1, W2, b2, w3, b3 = [torch.from_numpy(np.asarray(x, np.float64)) for x in w]
    h1 = torch.relu(X @ W1 + b1)
    h2 = torch.relu(h1 @ W2 + b2)
    return h1, h2, h2 @ w3 + b3, W2, w3


def exact(case, seed):
    if case["kind"] not in ("score", "train"):
        return None
    _, y, sign, rank = _flip_records(case["rows"], seed)
    X = _features64(sign, rank)
    w = _weights(seed)
    h1, h2, z, W2, w3 = _net64(w, X)
    if case["kind"] == "score":
        return h1, h2, z
    y, M = y.double(), case["rows"]
    loss = (torch.nn.functional.softplus(z) - y * z).mean().reshape(1)
    d3 = (torch.sigmoid(z) - y) / M
    d2 = d3[:, None] * w3 * (h2 > 0)
    d1 = (d2 @ W2.T) * (h1 > 0)
    pad = torch.zeros(3, dtype=torch.float64)
    grad = torch.cat([(d1.T @ X).reshape(-1), d1.sum(0), (d2.T @ h1).reshape(-1), d2.sum(0),
                      h2.T @ d3, d3.sum().reshape(1), pad])
    p0 = torch.cat([torch.from_numpy(x.T.reshape(-1).astype(np.float64)) for x in w] + [pad])
    m0, v0 = (x.double() for x in _moments(seed))
    m = 0.9 * m0 + 0.1 * grad
    v = 0.999 * v0 + 0.001 * grad * grad
    s = TRAIN_STEPS + 1
    par = p0 - 1e-3 * (m / (1 - 0.9 ** s)) / (torch.sqrt(v / (1 - 0.999 ** s)) + 1e-8)
    W2n = par[512 * 256 + 256:512 * 256 + 256 + 256 * 256]
    o3 = 512 * 256 + 256 + 256 * 256 + 256
    wbf = torch.cat([par[:512 * 256], W2n, W2n.reshape(256, 256).T.reshape(-1),
                     par[o3:o3 + 256]])
    return loss, grad, par, m, v, wbf
