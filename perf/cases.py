"""Performance cases of the kNN-graph library: what its callers have it do.

Every case is one pass through a public entry point on data resident in
device memory: exact k-NN (self, and queries against a larger set), NNDescent
(plain and encoder-seeded), encoder training, the UMAP fuzzy graph, PCA and
the embedding-quality metrics.  Sizes are those of the benchmark and the
tests: 5,000 / 20,011 / 1,000,000 x 50 Gaussian mixtures, the 70,000 x 784
pixel-like set, its 2-D embedding, and small calls of a few hundred rows.
Inputs are drawn on the device from the seed alone.
"""
from __future__ import annotations

import math

import torch

import paper_2603_04035_amd as knn

DEV = "cuda"
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


# ------------------------------------------------------------------ inputs

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * int(seed) + 17)
    return g


def _mixture(n, d, seed, comps=20):
    """Gaussian mixture with anisotropic components (scales over two octaves
    around 1, random linear maps), means ~ N(0, 4 I): the shape of the
    benchmark's 1,000,000 x 50 set."""
    g = _gen(seed)
    comps = max(1, min(comps, n // 20 + 1))
    mu = 2.0 * torch.randn(comps, d, generator=g, device=DEV)
    lab = torch.randint(0, comps, (n,), generator=g, device=DEV)
    X = torch.randn(n, d, generator=g, device=DEV)
    order = torch.argsort(lab, stable=True)
    cnt = torch.bincount(lab, minlength=comps).tolist()
    at = 0
    for c in range(comps):
        A = torch.randn(d, d, generator=g, device=DEV) / math.sqrt(d)
        s = torch.exp(torch.empty(d, device=DEV).uniform_(-1.15, 1.15, generator=g))
        rows = order[at:at + cnt[c]]
        X[rows] = (X[rows] * s) @ A
        at += cnt[c]
    return X + mu[lab]


def _pixels(n, d, seed, comps=10):
    """Image-like rows: ten prototypes with half of the pixels exactly 0,
    noise on the others, values on the 1/255 grid."""
    g = _gen(seed)
    field = torch.rand(comps, d, generator=g, device=DEV)
    mask = field > 0.5
    proto = torch.where(mask, 0.2 + 0.8 * torch.rand(comps, d, generator=g, device=DEV), 0.0)
    lab = torch.randint(0, comps, (n,), generator=g, device=DEV)
    X = torch.randn(n, d, generator=g, device=DEV).mul_(0.15).add_(proto[lab]).clamp_(0.0, 1.0)
    X = X.mul_(255.0).round_().div_(255.0)
    return X.mul_(mask[lab])


def _decaying(n, d, decay, seed):
    """Rows whose covariance eigenvalues fall as i^-decay (images' spectra
    fall like that), in a random basis, around a non-zero mean."""
    g = _gen(seed)
    s = torch.arange(1, d + 1, device=DEV, dtype=torch.float32).pow(-0.5 * decay)
    X = torch.randn(n, d, generator=g, device=DEV) * s
    for _ in range(4):   # random reflections: a cheap orthogonal change of basis
        v = torch.randn(d, generator=g, device=DEV)
        v /= v.norm()
        X -= 2.0 * (X @ v)[:, None] * v
    return X + torch.rand(d, generator=g, device=DEV)


def _rows(case, n, seed):
    f = _pixels if case.get("data") == "pixels" else _mixture
    return f(n, case["d"], seed).to(DTYPES[case.get("dtype", "f32")]).contiguous()


# ------------------------------------------------------------------- cases

def listed():
    return [
        # a few hundred rows: launches and latency are the call
        {"name": "exact-small", "op": "exact", "n": 500, "d": 50, "k": 15, "precision": "fp32"},
        # FP16-stored rows through the FP16 form, a ragged count (the FP16 tests' set)
        {"name": "exact-fp16-20k", "op": "exact", "n": 20011, "d": 50, "k": 15, "precision": "fp16", "dtype": "f16"},
        # the embedding's own neighbours, as the quality metrics need them
        {"name": "exact-2d", "op": "exact", "n": 70000, "d": 2, "k": 10, "precision": "fp32"},
        # the exact graph of the image-like set in full precision
        {"name": "exact-pixel-fp32", "op": "exact", "n": 70000, "d": 784, "k": 15, "precision": "fp32",
         "data": "pixels"},
        # the recall check: 10,000 sampled rows against the million they come from
        {"name": "query-1m", "op": "query", "n": 1_000_000, "nq": 10_000, "d": 50, "k": 15, "precision": "fp32"},
        # a small graph at the library's plain settings
        {"name": "nnd-5k", "op": "nnd", "n": 5000, "d": 50, "k": 15, "build_k": 15, "rho": 0.5, "iters": 8,
         "slots": 0, "rev": 0, "precision": "fp32", "init": "random"},
        # the headline build: 16-bit joins, seeded through an encoder
        {"name": "nnd-1m-seeded", "op": "nnd", "n": 1_000_000, "d": 50, "k": 15, "build_k": 30, "rho": 1.0,
         "iters": 30, "slots": 96, "rev": 30, "precision": "bf16", "init": "encoder"},
        # the plain form on wide rows
        {"name": "nnd-pixel-fp32", "op": "nnd", "n": 70000, "d": 784, "k": 15, "build_k": 31, "rho": 1.0,
         "iters": 30, "slots": 64, "rev": 31, "precision": "fp32", "init": "random", "data": "pixels"},
        # part of an encoder's training on the benchmark's 100,000-row sample
        {"name": "train-bf16", "op": "train", "n": 100_000, "d": 50, "k": 15, "batch": 4096, "steps": 50,
         "precision": "bf16"},
        # UMAP weights of the million-point graph
        {"name": "fuzzy-1m", "op": "fuzzy", "n": 1_000_000, "d": 50, "k": 15},
        # reduction to the pca_dim that comes before the graph
        {"name": "pca-70k", "op": "pca", "n": 70000, "d": 784, "p": 50, "decay": 1.2},
        # quality of a 2-D embedding of the image-like set
        {"name": "quality-70k", "op": "quality", "n": 70000, "d": 784, "e": 2, "k": 10, "data": "pixels"},
    ]


def _log(rng, lo, hi):
    """A whole number spread evenly over its logarithm, odd ones among them."""
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["exact", "exact", "query", "nnd", "nnd", "train", "fuzzy", "pca", "quality"])
    if op in ("exact", "query"):
        d = rng.choice([2, 3]) if rng.random() < 0.15 else _log(rng, 4, 784)
        c = {"op": op, "n": _log(rng, 300, 70000), "d": d, "k": rng.randint(5, 16),
             "precision": rng.choice(["fp32", "fp32", "bf16", "fp16"]), "dtype": rng.choice(["f32", "f32", "f16", "bf16"]),
             "data": rng.choice(["mixture", "pixels"] if d > 64 else ["mixture"])}
        if op == "query":
            c["n"] = _log(rng, 1000, 1_000_000)
            c["nq"] = min(c["n"], _log(rng, 50, 10_000))
            c["n"] = min(c["n"], 50_000_000 // d)
            c["nq"] = min(c["nq"], c["n"])
        return c
    if op == "nnd":
        d = _log(rng, 8, 784)
        n = min(_log(rng, 1000, 1_000_000), 50_000_000 // d)
        rho = rng.choice([0.5, 1.0])
        K = rng.randint(15, 31)
        s = math.ceil(rho * K)
        return {"op": "nnd", "n": n, "d": d, "k": rng.randint(8, 15), "build_k": K, "rho": rho,
                "iters": rng.choice([8, 20, 30]), "slots": rng.choice([0, 64, 96]), "rev": rng.choice([0, s]),
                "precision": rng.choice(["fp32", "bf16", "fp16"]), "init": rng.choice(["random", "encoder"]),
                "dtype": rng.choice(["f32", "f32", "f16"]), "data": "pixels" if d > 64 and rng.random() < 0.5 else "mixture"}
    if op == "train":
        return {"op": "train", "n": _log(rng, 2000, 100_000), "d": _log(rng, 20, 784), "k": rng.randint(8, 15),
                "batch": _log(rng, 128, 4096), "steps": rng.randint(5, 50), "precision": rng.choice(["fp32", "bf16"])}
    if op == "fuzzy":
        return {"op": "fuzzy", "n": _log(rng, 1000, 1_000_000), "d": rng.choice([20, 50]), "k": rng.randint(5, 30)}
    if op == "pca":
        d = _log(rng, 20, 784)
        return {"op": "pca", "n": _log(rng, 3000, 70000), "d": d, "p": rng.randint(2, min(d, 64)),
                "decay": rng.choice([0.8, 1.0, 1.2, 1.5])}
    return {"op": "quality", "n": _log(rng, 500, 70000), "d": _log(rng, 8, 784), "e": rng.choice([2, 2, 3, 20]),
            "k": rng.randint(5, 16), "data": rng.choice(["mixture", "pixels"])}


# ----------------------------------------------------------------- prepare

def _graph(X, k, seed):
    """A k-NN graph of X as the pipeline hands it on: exact when small, NNDescent's else."""
    if X.shape[0] <= 100_000:
        return knn.knn_exact(X, k)
    idx, dist, _ = knn.nndescent_build(X, k, seed=seed, precision="bf16", build_k=min(32, max(k, 30)),
                                       sample_rate=1.0, cand_slots=96)
    return idx, dist


def prepare(case, seed):
    op, n = case["op"], case["n"]
    s = {"case": case}
    if op == "pca":
        s["X"] = _decaying(n, case["d"], case["decay"], seed)
        return s
    if op == "fuzzy":
        # one graph per size, its points numbered and its rows' distances
        # scaled by the seed: the union then has as many entries for each seed
        idx, dist = _graph(_mixture(n, case["d"], 0), case["k"], 0)
        g = _gen(seed + 3)
        new = torch.randperm(n, generator=g, device=DEV)
        s["idx"], s["dist"] = torch.empty_like(idx), torch.empty_like(dist)
        s["idx"][new] = new[idx.long()].to(torch.int32)
        s["dist"][new] = dist * torch.empty(n, 1, device=DEV).uniform_(0.8, 1.25, generator=g)
        return s
    s["X"] = X = _rows(case, n, seed)
    if op == "query":
        # sampled rows of the set itself, each excluding itself
        rows = torch.randperm(n, generator=_gen(seed + 5), device=DEV)[:case["nq"]].sort().values
        s["Q"], s["self"] = X[rows].contiguous(), rows.to(torch.int32)
    elif op == "nnd":
        s["opts"] = dict(precision=case["precision"], build_k=case["build_k"], sample_rate=case["rho"],
                         max_iters=case["iters"], cand_slots=case["slots"], rev_slots=case["rev"], seed=seed)
        if case["init"] == "encoder":
            s["enc"] = knn.Encoder(case["d"], seed=1)
            s["opts"].update(init_kind="encoder", encoder=s["enc"], proj_count=4, proj_window=8)
    elif op == "train":
        s["enc"] = knn.Encoder(case["d"], seed=seed % 1000)
        s["weights"] = s["enc"].get_weights()
        s["graph"], _ = _graph(X, case["k"], seed)
    elif op == "quality":
        g = _gen(seed + 9)
        R = torch.randn(case["d"], case["e"], generator=g, device=DEV)
        s["Y"] = (X.float() @ R + 0.5 * torch.randn(n, case["e"], generator=g, device=DEV)).contiguous()
    return s


# --------------------------------------------------------------------- run

def run(s):
    c = s["case"]
    op = c["op"]
    if op == "exact":
        return knn.knn_exact(s["X"], c["k"], precision=c["precision"])
    if op == "query":
        return knn.knn_exact_query(s["Q"], s["X"], c["k"], q_self=s["self"], precision=c["precision"])
    if op == "nnd":
        idx, dist, st = knn.nndescent_build(s["X"], c["k"], **s["opts"])
        return idx, dist, st["iters"]
    if op == "train":
        # a training run from given weights; the trained weights come back
        s["enc"].set_weights(*s["weights"])
        loss = s["enc"].train(s["X"], s["graph"], steps=c["steps"], batch=c["batch"], lr=2e-3, seed=3,
                              precision=c["precision"])
        return [loss, *s["enc"].get_weights()]
    if op == "fuzzy":
        return knn.fuzzy_graph(s["idx"], s["dist"])
    if op == "pca":
        return knn.pca(s["X"], c["p"])
    return knn.quality(s["X"], s["Y"], c["k"], per_row=True)


# -------------------------------------------------------------------- work

def work(case):
    """Each input read once, each output written once; products that the
    definition needs (pairwise distances, the Gram, the layers)."""
    op, n, d, k = case["op"], case["n"], case.get("d", 0), case.get("k", 0)
    eb = 4 if case.get("dtype", "f32") == "f32" else 2
    if op in ("exact", "query"):
        nq = case.get("nq", n)
        return {"bytes": n * d * eb + nq * k * 8 + (nq * d * eb if op == "query" else 0), "flops": 2.0 * nq * n * d}
    if op == "nnd":
        # a build that knew each point's neighbours would still form their distances
        return {"bytes": n * d * eb + n * k * 8, "flops": 3.0 * n * k * d}
    if op == "train":
        P = d * 64 + 64 * 32
        return {"bytes": case["steps"] * (3 * case["batch"] * d * eb + 6 * P * 4),
                "flops": 6.0 * case["steps"] * 3 * case["batch"] * P}
    if op == "fuzzy":
        return {"bytes": n * k * 8 + n * 8 + n * k * 4 + n * 8 + 1.5 * n * k * 8, "flops": 10.0 * n * k}
    if op == "pca":
        return {"bytes": n * d * 4 + n * case["p"] * 4, "flops": float(n) * d * (d + 1) + 2.0 * n * d * case["p"]}
    return {"bytes": n * (d + case["e"]) * 4 + n * 20, "flops": 2.0 * n * n * (d + case["e"])}


# ------------------------------------------------------------------- exact

def _knn64(Q, R, k, self_rows):
    """The k smallest FP64 distances of each row of Q to the rows of R."""
    R64 = R.double()
    rn = (R64 * R64).sum(1)
    step = max(1, min(2048, 200_000_000 // R.shape[0]))
    out = []
    for a in range(0, Q.shape[0], step):
        q = Q[a:a + step].double()
        D = rn[None, :] + (q * q).sum(1)[:, None] - 2.0 * (q @ R64.T)
        sr = self_rows[a:a + step].long()
        D[torch.arange(len(q), device=DEV), sr] = float("inf")
        j = torch.topk(D, min(D.shape[1], k + 4), largest=False).indices   # then without the expansion
        e = torch.stack([((R64[j[:, t]] - q) ** 2).sum(1) for t in range(j.shape[1])], 1)
        e = torch.where(j == sr[:, None], float("inf"), e)
        out.append(e.sort(1).values[:, :k].sqrt())
    return torch.cat(out)


def _quality64(X, Y, k):
    n = X.shape[0]
    X, Y = X.double(), Y.double()
    xn, yn = (X * X).sum(1), (Y * Y).sum(1)
    hits = trust = cont = 0
    step = max(1, min(1024, 100_000_000 // n))
    for a in range(0, n, step):
        b = min(n, a + step)
        i = torch.arange(b - a, device=DEV)
        D = [xn[None, :] + xn[a:b, None] - 2.0 * (X[a:b] @ X.T)]
        if Y.shape[1] <= 3:
            D.append(sum((Y[None, :, t] - Y[a:b, t, None]) ** 2 for t in range(Y.shape[1])))
        else:
            D.append(yn[None, :] + yn[a:b, None] - 2.0 * (Y[a:b] @ Y.T))
        for m in D:
            m[i, i + a] = float("inf")
        N, L = (torch.topk(m, k, largest=False).indices for m in D)
        hits += int((N[:, :, None] == L[:, None, :]).sum())
        for t in range(k):
            r = (D[0] < D[0][i, L[:, t]][:, None]).sum(1) + 1 - k
            trust += int(r.clamp_min(0).sum())
            r = (D[1] < D[1][i, N[:, t]][:, None]).sum(1) + 1 - k
            cont += int(r.clamp_min(0).sum())
    z = 2.0 / (float(n) * k * (2.0 * n - 3.0 * k - 1.0))
    return (hits / (float(n) * k), 1.0 - z * trust, 1.0 - z * cont)


def _fuzzy64(idx, dist):
    n, k = idx.shape
    d = dist.double()
    big = torch.where(d > 0, d, float("inf")).min(1).values
    rho = torch.where(torch.isfinite(big), big, 0.0)
    x = (d - rho[:, None]).clamp_min(0.0)
    target = math.log2(k)
    has = (x == 0).sum(1) < target
    lo, hi = torch.zeros(n, dtype=torch.float64, device=DEV), x.max(1).values.clamp_min(1e-300)
    for _ in range(60):
        hi = torch.where(torch.exp(-x / hi[:, None]).sum(1) < target, 2.0 * hi, hi)
    for _ in range(90):
        mid = 0.5 * (lo + hi)
        low = torch.exp(-x / mid[:, None]).sum(1) < target
        lo, hi = torch.where(low, mid, lo), torch.where(low, hi, mid)
    sigma = torch.where(has, 0.5 * (lo + hi), 0.0)
    w = torch.where(has[:, None], torch.exp(-x / sigma.clamp_min(1e-300)[:, None]), (x == 0).double())
    i = torch.arange(n, device=DEV)[:, None].expand(n, k).reshape(-1)
    j, v = idx.reshape(-1).long(), w.reshape(-1)
    key, at = torch.unique(torch.cat([i * n + j, j * n + i]), return_inverse=True)
    a = torch.zeros(len(key), dtype=torch.float64, device=DEV).index_put_((at[:n * k],), v)
    b = torch.zeros(len(key), dtype=torch.float64, device=DEV).index_put_((at[n * k:],), v)
    return [rho, sigma, w, None, None, a + b - a * b]


def _pca64(X, p):
    X = X.double()
    mu = X.mean(0)
    X = X - mu
    w, V = torch.linalg.eigh((X.T @ X / (X.shape[0] - 1)).cpu())
    w, V = w.flip(0)[:p].to(DEV), V.flip(1)[:, :p].to(DEV)
    top = V.abs().argmax(0)
    V = V * torch.sign(V[top, torch.arange(p, device=DEV)])
    return [X @ V, V, w, mu]


def exact(case, seed):
    op = case["op"]
    if op in ("nnd", "train"):
        # an approximate graph has no value of its own, and a training run's
        # triplets are the library's draws
        return None
    s = prepare(case, seed)
    if op == "exact":
        return [None, _knn64(s["X"], s["X"], case["k"], torch.arange(case["n"], device=DEV))]
    if op == "query":
        return [None, _knn64(s["Q"], s["X"], case["k"], s["self"])]
    if op == "fuzzy":
        return _fuzzy64(s["idx"], s["dist"])
    if op == "pca":
        return _pca64(s["X"], case["p"])
    return [list(_quality64(s["X"], s["Y"], case["k"])), [None, None, None]]
