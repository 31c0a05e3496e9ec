"""The work that users of this framework have it do, as cases that can be timed.

A case is one pass through the public entry points (Plan.sweep, Plan.half,
Plan.mu_sweep, Plan.foldin, and a training step of the warm-start network) on
inputs made from a seed: Zipf bag-of-words corpora in CSR, parts-based dense
images, new documents for fold-in.  `listed()` names the cases, `draw()` gives
further ones of the same ranges, `prepare()` makes what a program holds before
the call, `run()` is the call, `work()` its compulsory bytes and operations and
`exact()` the same result in 64 bits.
"""
import math

import numpy as np
import torch

from paper_1904_07935_amd.api import Matrix, Mlp, Plan

DEV = "cuda"
EPS = 1e-16
LR = 1e-3


def listed():
    return [
        # the smallest factorisation (the parity problem's size): launches and latency
        {"name": "dense-small", "kind": "sweep", "fmt": "dense", "prec": "fp32",
         "V": 1000, "D": 800, "K": 16, "obj": False},
        # a 20 Newsgroups sized corpus
        {"name": "bow-20news", "kind": "sweep", "fmt": "csr", "prec": "fp32",
         "V": 26000, "D": 11000, "K": 200, "len": 77, "obj": False},
        # a small corpus with odd sizes and rank, watched by its objective
        {"name": "bow-ragged", "kind": "sweep", "fmt": "csr", "prec": "fp32",
         "V": 6037, "D": 2741, "K": 77, "len": 60, "obj": True},
        # a dense image set
        {"name": "faces", "kind": "sweep", "fmt": "dense", "prec": "fp32",
         "V": 10000, "D": 10000, "K": 240, "obj": False},
        # the same with BF16 products: the W half
        {"name": "faces-W-bf16", "kind": "half_W", "fmt": "dense", "prec": "bf16",
         "V": 10000, "D": 10000, "K": 240},
        # the large corpus: both halves of its sweep, and the H half with BF16 products
        {"name": "large-H", "kind": "half_H", "fmt": "csr", "prec": "fp32",
         "V": 100000, "D": 300000, "K": 400, "len": 99},
        {"name": "large-W", "kind": "half_W", "fmt": "csr", "prec": "fp32",
         "V": 100000, "D": 300000, "K": 400, "len": 99},
        {"name": "large-H-bf16", "kind": "half_H", "fmt": "csr", "prec": "bf16",
         "V": 100000, "D": 300000, "K": 400, "len": 99},
        # the multiplicative-update baseline on images
        {"name": "images-mu", "kind": "mu", "fmt": "dense", "prec": "fp32",
         "V": 4096, "D": 3001, "K": 100},
        # a batch of new documents, started by the network
        {"name": "foldin-batch", "kind": "foldin", "init": "mlp", "docs": 100000, "V": 26000,
         "K": 200, "len": 77, "sweeps": 2, "trace": False, "hidden": 512},
        # a handful of new documents in a serving loop, objective reported
        {"name": "foldin-serve", "kind": "foldin", "init": "wta", "docs": 256, "V": 26000,
         "K": 100, "len": 77, "sweeps": 5, "trace": True, "hidden": 0},
        # one minibatch of the network's training: forward, backward, Adam
        {"name": "train-step", "kind": "train", "batch": 1024, "K": 200, "hidden": 512},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["sweep_dense", "sweep_csr", "sweep_csr", "half", "half_dense", "mu",
                       "foldin", "foldin", "train"])
    if kind == "sweep_dense":
        V, D = _log(rng, 800, 10000), _log(rng, 800, 10000)
        return {"kind": "sweep", "fmt": "dense", "prec": "fp32", "V": V, "D": D,
                "K": _log(rng, 8, 240), "obj": rng.random() < 0.3}
    if kind == "sweep_csr":
        return {"kind": "sweep", "fmt": "csr", "prec": "fp32", "V": _log(rng, 4000, 60000),
                "D": _log(rng, 2500, 60000), "K": _log(rng, 16, 400),
                "len": rng.randint(40, 99), "obj": rng.random() < 0.3}
    if kind == "half":
        which, prec = rng.choice([("half_H", "fp32"), ("half_W", "fp32"), ("half_H", "bf16")])
        return {"kind": which, "fmt": "csr", "prec": prec, "V": _log(rng, 20000, 100000),
                "D": _log(rng, 20000, 300000), "K": _log(rng, 60, 400),
                "len": rng.randint(60, 99)}
    if kind == "half_dense":
        return {"kind": rng.choice(["half_H", "half_W"]), "fmt": "dense", "prec": "bf16",
                "V": _log(rng, 1500, 10000), "D": _log(rng, 1500, 10000), "K": _log(rng, 30, 240)}
    if kind == "mu":
        return {"kind": "mu", "fmt": "dense", "prec": "fp32", "V": _log(rng, 1000, 6000),
                "D": _log(rng, 1000, 6000), "K": _log(rng, 16, 200)}
    if kind == "foldin":
        init = rng.choice(["wta", "mlp"])
        return {"kind": "foldin", "init": init, "docs": _log(rng, 32, 100000), "V": 26000,
                "K": _log(rng, 20, 240), "len": rng.randint(40, 99), "sweeps": rng.randint(1, 5),
                "trace": rng.random() < 0.5, "hidden": 512 if init == "mlp" else 0}
    return {"kind": "train", "batch": _log(rng, 200, 4096), "K": _log(rng, 20, 240),
            "hidden": rng.choice([128, 256, 512])}


# ------------------------------------------------------------- inputs ----

def _gen(seed, salt):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000003 + salt)


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _bow(case, docs, seed, term_major):
    """A bag-of-words matrix: Zipf term popularity, tf-idf values, unit-norm
    documents.  Returns int32 rowptr, int32 col, float32 val of the CSR with a row
    per term (term_major) or per document."""
    V = case["V"]
    g = _gen(seed, 1)
    s = 1.1 if V < 60000 else 1.05
    p = torch.arange(1, V + 1, dtype=torch.float64, device=DEV).pow(-s)
    cdf = torch.cumsum(p, 0)
    cdf = (cdf / cdf[-1]).float()
    perm = torch.argsort(_rand(g, V))
    tokens = 1 + torch.poisson(torch.full((docs,), 1.5 * case["len"], device=DEV), generator=g).long()
    doc = torch.repeat_interleave(torch.arange(docs, device=DEV), tokens)
    rank = torch.searchsorted(cdf, _rand(g, doc.numel())).clamp_(max=V - 1)
    key = perm[rank] * docs + doc if term_major else doc * V + perm[rank]
    key, count = torch.unique(key, return_counts=True)
    row = key // (docs if term_major else V)
    col = key - row * (docs if term_major else V)
    term, doc = (row, col) if term_major else (col, row)
    df = torch.bincount(term, minlength=V)
    idf = torch.log((1.0 + docs) / (1.0 + df.double())) + 1.0
    x = count.double() * idf[term]
    sq = torch.zeros(docs, dtype=torch.int64, device=DEV)  # fixed point: the same in any order
    sq.index_add_(0, doc, (x * x * 2.0 ** 24).round().long())
    val = (x / torch.sqrt(sq[doc].double() / 2.0 ** 24)).float()
    rows = V if term_major else docs
    ptr = torch.zeros(rows + 1, dtype=torch.int32, device=DEV)
    ptr[1:] = torch.cumsum(torch.bincount(row, minlength=rows), 0).int()
    return ptr, col.int().contiguous(), val.contiguous()


def _images(case, seed):
    """Dense parts-based data and factors in mid-run: A = W0 H0 + noise with sparse
    non-negative W0, H0, and both factors some way off."""
    V, D, K = case["V"], case["D"], case["K"]
    g = _gen(seed, 2)

    def part(n):
        x = torch.randn(n, K, generator=g, device=DEV).abs_()
        return x * (_rand(g, n, K) < 0.25)

    W0, H0 = part(V), part(D)
    A = W0 @ H0.T
    A += 0.05 * _rand(g, V, D)
    W = W0 * (0.5 + _rand(g, V, K)) + 1e-3 * _rand(g, V, K)
    H = H0 * (0.5 + _rand(g, D, K)) + 1e-3 * _rand(g, D, K)
    H *= torch.sqrt((W.double() ** 2).sum(0)).float()
    return A.contiguous(), W.contiguous(), H.contiguous()


def _bow_start(case, val, seed):
    """The usual random start of a corpus: U[0,1) factors, H scaled to the data's mean."""
    V, D, K = case["V"], case["D"], case["K"]
    g = _gen(seed, 3)
    mean = float(val.double().sum()) / (V * D)
    h = mean * math.sqrt(V / 3.0) / (0.25 * K)
    return _rand(g, V, K), _rand(g, D, K) * h


def _problem(case, seed):
    """(A dense or None, CSR or None, W, Ht) of a factorisation case."""
    if case["fmt"] == "dense":
        A, W, Ht = _images(case, seed)
        return A, None, W, Ht
    csr = _bow(case, case["D"], seed, True)
    W, Ht = _bow_start(case, csr[2], seed)
    return None, csr, W, Ht


def _model(case, seed):
    """A fitted topic matrix (few heavy terms per topic) and the corpus that a fold-in
    plan was made from."""
    V, K = case["V"], case["K"]
    fit = dict(case, D=max(2 * K, 512))
    csr = _bow(fit, fit["D"], seed + 77, True)
    g = _gen(seed, 4)
    return fit["D"], csr, _rand(g, V, K).pow(6), _rand(g, fit["D"], K)


def _network(case, seed):
    K, H = case["K"], case["hidden"]
    r = np.random.default_rng([int(seed), 5])

    def u(fan, *shape):
        return ((2.0 * r.random(shape) - 1.0) / math.sqrt(fan)).astype(np.float32)

    return {"W1": u(K, H, K), "b1": u(K, H), "W2": u(H, K, H), "b2": u(H, K)}


def _batch(case, seed):
    g = _gen(seed, 6)
    X = _rand(g, case["batch"], case["K"]).pow(4)
    X /= X.norm(dim=1, keepdim=True)
    Y = _rand(g, case["batch"], case["K"]).pow(8)
    return X.contiguous(), Y.contiguous()


def prepare(case, seed):
    kind = case["kind"]
    if kind == "train":
        net = Mlp(case["K"], case["hidden"], DEV, seed=None)
        net.set_masters(_network(case, seed))
        X, Y = _batch(case, seed)
        return {"kind": kind, "net": net, "X": X, "Y": Y}
    if kind == "foldin":
        D, (ptr, col, val), W, Ht = _model(case, seed)
        plan = Plan(Matrix(case["V"], D, rowptr=ptr, col=col, val=val), W, Ht, eps=EPS)
        net = None
        if case["init"] == "mlp":
            net = Mlp(case["K"], case["hidden"], DEV, seed=None)
            net.set_masters(_network(case, seed))
        ptr, col, val = _bow(case, case["docs"], seed, False)
        new = Matrix(case["docs"], case["V"], rowptr=ptr, col=col, val=val)
        return {"kind": kind, "plan": plan, "net": net, "new": new, "init": case["init"],
                "sweeps": case["sweeps"], "trace": case["trace"],
                "H": torch.empty(case["docs"], case["K"], device=DEV)}
    A, csr, W, Ht = _problem(case, seed)
    if A is not None:
        M = Matrix(case["V"], case["D"], dense=A)
    else:
        M = Matrix(case["V"], case["D"], rowptr=csr[0], col=csr[1], val=csr[2])
    plan = Plan(M, W, Ht, eps=EPS, precision=case["prec"])
    if kind == "half_W" and csr is not None:
        plan.half("H")  # the W half follows the H half of the same sweep
    return {"kind": kind, "plan": plan, "obj": case.get("obj", False)}


def run(s):
    kind = s["kind"]
    if kind == "train":
        loss, grads, flat = s["net"].loss_grad(s["X"], s["Y"])
        s["net"].adam_step(flat, lr=LR)
        return {"loss": loss, "grads": grads, "weights": s["net"].masters()}
    plan = s["plan"]
    if kind == "foldin":
        tr = plan.foldin(s["new"], s["H"], init=s["init"], mlp=s["net"], n_sweeps=s["sweeps"],
                         trace=s["trace"])
        return {"H": s["H"], "trace": tr}
    if kind == "half_H":
        plan.half("H")
        return {"Ht": plan.Ht}
    if kind == "half_W":
        plan.half("W")
        return {"W": plan.W}
    if kind == "mu":
        plan.mu_sweep(1)
        return {"W": plan.W, "Ht": plan.Ht}
    rel = plan.sweep(1, objective=s["obj"])
    return {"W": plan.W, "Ht": plan.Ht, "rel": rel}


# --------------------------------------------------------- work and oracle ----

def work(case):
    K = case["K"]
    if case["kind"] == "train":
        B, H = case["batch"], case["hidden"]
        n = 2 * H * K + H + K
        return {"bytes": 4.0 * (2 * B * K + n * (1 + 3 * 2)), "flops": 2.0 * B * K * H * 5 + 12.0 * n}
    if case["kind"] == "foldin":
        d, V = case["docs"], case["V"]
        nnz = float(d * case["len"])
        return {"bytes": 8.0 * nnz + 4.0 * (V * K + d * K),
                "flops": 2.0 * nnz * K + 2.0 * V * K * K + 2.0 * d * K * K * case["sweeps"]
                + 4.0 * d * K * case["hidden"]}
    V, D = case["V"], case["D"]
    dense = case["fmt"] == "dense"
    nnz = float(V * D) if dense else float(D * case["len"])
    el = 2.0 if case["prec"] == "bf16" else 4.0
    a_bytes = nnz * (el if dense else el + 4.0)
    factors = 4.0 * K * (V + D)
    if case["kind"] == "half_H":
        return {"bytes": a_bytes + factors + 4.0 * D * K,
                "flops": 2.0 * nnz * K + 2.0 * V * K * K + 2.0 * D * K * K}
    if case["kind"] == "half_W":
        return {"bytes": a_bytes + factors + 4.0 * V * K,
                "flops": 2.0 * nnz * K + 2.0 * D * K * K + 2.0 * V * K * K}
    obj = 2.0 * V * D * K if case.get("obj") and dense else 0.0
    return {"bytes": a_bytes + 2.0 * factors,
            "flops": 4.0 * nnz * K + 4.0 * (V + D) * K * K + obj}


def _spmm64(ptr, col, val, X):
    """CSR times X in 64 bits."""
    n = ptr.numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEV), (ptr[1:] - ptr[:-1]).long())
    out = torch.zeros(n, X.shape[1], dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // X.shape[1])
    for a in range(0, col.numel(), step):
        b = min(a + step, col.numel())
        out.index_add_(0, row[a:b], X[col[a:b].long()] * val[a:b].double()[:, None])
    return out


def _spmm64_t(ptr, col, val, X, cols):
    """The transposed CSR times X in 64 bits."""
    n = ptr.numel() - 1
    row = torch.repeat_interleave(torch.arange(n, device=DEV), (ptr[1:] - ptr[:-1]).long())
    out = torch.zeros(cols, X.shape[1], dtype=torch.float64, device=DEV)
    step = max(1, (1 << 28) // X.shape[1])
    for a in range(0, col.numel(), step):
        b = min(a + step, col.numel())
        out.index_add_(0, col[a:b].long(), X[row[a:b]] * val[a:b].double()[:, None])
    return out


def _h_loop(H, R, S):
    for k in range(H.shape[1]):
        H[:, k] = torch.clamp(H[:, k] + R[:, k] - H @ S[:, k], min=EPS)


def _w_loop(W, P, Q):
    for k in range(W.shape[1]):
        u = torch.clamp(W[:, k] * Q[k, k] + P[:, k] - W @ Q[:, k], min=EPS)
        W[:, k] = u / u.norm()


def _gelu(z):
    return 0.5 * z * (1.0 + torch.erf(z / math.sqrt(2.0)))


def _exact_train(case, seed):
    p = {k: torch.tensor(v, dtype=torch.float64, device=DEV) for k, v in _network(case, seed).items()}
    X, Y = (t.double() for t in _batch(case, seed))
    z1 = X @ p["W1"].T + p["b1"]
    a1 = _gelu(z1)
    z2 = a1 @ p["W2"].T + p["b2"]
    d = torch.nn.functional.softplus(z2) - Y
    loss = (d * d).mean()
    dz2 = 2.0 / d.numel() * d * torch.sigmoid(z2)
    cdf = 0.5 * (1.0 + torch.erf(z1 / math.sqrt(2.0)))
    pdf = torch.exp(-0.5 * z1 * z1) / math.sqrt(2.0 * math.pi)
    dz1 = (dz2 @ p["W2"]) * (cdf + z1 * pdf)
    grads = {"W1": dz1.T @ X, "b1": dz1.sum(0), "W2": dz2.T @ a1, "b2": dz2.sum(0)}
    weights = {k: p[k] - LR * g / (g.abs() + 1e-8) for k, g in grads.items()}  # Adam's first step
    return {"loss": loss.reshape(()), "grads": grads, "weights": weights}


def _exact_foldin(case, seed):
    _, _, W, _ = _model(case, seed)
    W = W.double()
    W /= W.norm(dim=0)
    csr = _bow(case, case["docs"], seed, False)
    R, S = _spmm64(*csr, W), W.T @ W
    if case["init"] == "wta":
        H = R.clamp(min=EPS)
    else:
        p = {k: torch.tensor(v, dtype=torch.float64, device=DEV)
             for k, v in _network(case, seed).items()}
        n = R.norm(dim=1, keepdim=True)
        x = torch.where(n > 0, R / n, torch.zeros_like(R))
        y = torch.nn.functional.softplus(_gelu(x @ p["W1"].T + p["b1"]) @ p["W2"].T + p["b2"])
        H = (n * y).clamp(min=EPS)
    a2 = (csr[2].double() ** 2).sum()

    def rel():
        return torch.sqrt((a2 - 2.0 * (H * R).sum() + ((H.T @ H) * S).sum()) / a2)

    trace = [rel()]
    for _ in range(case["sweeps"]):
        _h_loop(H, R, S)
        trace.append(rel())
    return {"H": H, "trace": trace if case["trace"] else None}


def exact(case, seed):
    kind = case["kind"]
    if kind == "train":
        return _exact_train(case, seed)
    if kind == "foldin":
        return _exact_foldin(case, seed)
    A, csr, W, H = _problem(case, seed)
    W, H = W.double(), H.double()
    W /= W.norm(dim=0)
    A = None if A is None else A.double()

    def prod_r():
        return A.T @ W if A is not None else _spmm64_t(*csr, W, case["D"])

    def prod_p():
        return A @ H if A is not None else _spmm64(*csr, H)

    if kind == "mu":
        H = H * prod_r() / (H @ (W.T @ W) + EPS)
        W = W * prod_p() / (W @ (H.T @ H) + EPS)
        return {"W": W, "Ht": H}
    if kind != "half_W" or csr is not None:
        _h_loop(H, prod_r(), W.T @ W)
    if kind == "half_H":
        return {"Ht": H}
    P = prod_p()
    _w_loop(W, P, H.T @ H)
    if kind == "half_W":
        return {"W": W}
    rel = None
    if case["obj"]:
        if A is not None:
            a2, e2 = (A * A).sum(), ((A - W @ H.T) ** 2).sum()
        else:
            a2 = (csr[2].double() ** 2).sum()
            e2 = a2 - 2.0 * (W * P).sum() + ((W.T @ W) * (H.T @ H)).sum()
        rel = [torch.sqrt(e2 / a2)]
    return {"W": W, "Ht": H, "rel": rel}
