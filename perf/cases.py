"""The work that users of this library have it do, as measurable cases.

A case is one public call (or the loop behind one) at sizes taken from the
library's workloads and tests:

* ``fit``      kkm_fit_ex end to end on a small problem: launch latency counts.
* ``step``     one reassignment step on a K already in memory, dense or
               strip-packed, float32 or bfloat16.
* ``gram``     the kernel matrix, dense or strip-packed, for each arithmetic
               of the product and each storage type.
* ``matfree``  one step that recomputes the kernel values.
* ``batched``  many uneven problems in one call.
* ``train``    training steps of the feature network on fresh batches.
* ``warm``     the learned warm start: features, seeding, Lloyd.

Points are equal-weight mixtures in R^d (means N(0, 1), spread 0.25) as in the
mixture workloads, or the [0, 1]-valued, mostly zero points of the MNIST-shaped
one.  Labels that enter a step are the generating components with a part of
them redrawn, as in the middle of a run: clusters differ clearly, so the
labels that come out do not hang on the last bit of a distance.  The objective
is a sum of float32 distances: where the distances themselves come back it is
not returned beside them, and a fit's objective is returned in float32.
"""
import math

import numpy as np
import torch

import paper_2501_05587_amd as kkm

W = 1024  # columns of a strip of the packed layout
PREC = {"f32": kkm.F32, "bf16": kkm.BF16, "fp8": kkm.FP8_ROWSCALED}
KERNEL = {"gauss": kkm.GAUSS, "poly": kkm.POLY, "linear": kkm.LINEAR}


def listed():
    return [
        # the smallest whole call: the rings workload's size, 30 fixed iterations (the paper's protocol)
        {"name": "fit_1k", "what": "fit", "n": 1000, "d": 16, "k": 4, "iters": 30},
        # a single step as a serving loop calls it: a few strips, ragged
        {"name": "step_dense_f32_3k", "what": "step", "layout": "dense", "store": "f32", "n": 3001, "k": 12},
        # the paper's MNIST-shaped workload: one iteration, float32 K
        {"name": "step_dense_f32_60k", "what": "step", "layout": "dense", "store": "f32", "n": 60000, "k": 10},
        # the headline's form of the step (strip-packed float32 K, k = 64) at half its points
        {"name": "step_packed_f32_100k", "what": "step", "layout": "packed", "store": "f32", "n": 100000, "k": 64},
        # the learned workload's refinement: strip-packed bfloat16 K, k = 32
        {"name": "step_packed_bf16_100k", "what": "step", "layout": "packed", "store": "bf16", "n": 100000, "k": 32},
        # the MNIST-shaped kernel matrix: float32 product, polynomial
        {"name": "gram_f32_60k", "what": "gram", "prec": "f32", "layout": "dense", "store": "f32", "kernel": "poly", "n": 60000, "d": 784},
        # the mixed form's kernel matrix: bfloat16 product, strip-packed bfloat16 K, d = 1024
        {"name": "gram_bf16_packed_100k", "what": "gram", "prec": "bf16", "layout": "packed", "store": "bf16", "kernel": "gauss", "n": 100000, "d": 1024},
        # the FP8 product on a ragged mid-size problem
        {"name": "gram_fp8_20k", "what": "gram", "prec": "fp8", "layout": "dense", "store": "bf16", "kernel": "gauss", "n": 20011, "d": 256},
        # a step without a stored K, for memory
        {"name": "matfree_bf16_50k", "what": "matfree", "prec": "bf16", "kernel": "gauss", "n": 50021, "d": 128, "k": 32},
        # uneven problems in shared launches, as the batched workload draws them
        {"name": "batched_48", "what": "batched", "prec": "bf16", "store": "f32", "count": 48, "nmin": 256, "nmax": 8192, "iters": 30},
        # the feature network's training, in batches of 64 as the learned workload trains it
        {"name": "train_d128", "what": "train", "d": 128, "B": 64, "steps": 16},
        # the learned warm start: d and k of the learned workload, half its points
        {"name": "warm_50k", "what": "warm", "n": 50000, "d": 128, "k": 32, "restarts": 4, "iters": 20},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["fit", "step", "step", "step", "gram", "gram", "gram", "matfree", "batched", "train", "warm"])
    if what == "fit":
        return {"what": what, "n": _log(rng, 300, 4000), "d": _log(rng, 16, 256), "k": rng.randint(2, 10), "iters": 30}
    if what == "step":
        layout = rng.choice(["dense", "packed"])
        return {"what": what, "layout": layout, "store": rng.choice(["f32", "bf16"]),
                "n": _log(rng, 1000, 60000 if layout == "dense" else 100000), "k": _log(rng, 2, 100)}
    if what == "gram":
        prec = rng.choice(["f32", "f32", "bf16", "fp8"])
        return {"what": what, "prec": prec, "layout": rng.choice(["dense", "packed"]),
                "store": "f32" if prec == "f32" else rng.choice(["f32", "bf16"]),
                "kernel": rng.choice(["gauss", "gauss", "poly", "linear"]),
                "n": _log(rng, 1000, 60000), "d": _log(rng, 16, 784)}
    if what == "matfree":
        return {"what": what, "prec": rng.choice(["f32", "bf16", "fp8"]), "kernel": rng.choice(["gauss", "poly"]),
                "n": _log(rng, 2000, 50000), "d": _log(rng, 16, 256), "k": _log(rng, 2, 64)}
    if what == "batched":
        return {"what": what, "prec": rng.choice(["f32", "bf16"]), "store": rng.choice(["f32", "bf16"]),
                "count": _log(rng, 4, 48), "nmin": 256, "nmax": _log(rng, 1000, 8192), "iters": 30}
    if what == "train":
        return {"what": what, "d": _log(rng, 16, 1024), "B": rng.choice([64, 128, 256]), "steps": rng.randint(4, 16)}
    return {"what": what, "n": _log(rng, 2000, 50000), "d": _log(rng, 16, 256), "k": rng.randint(2, 32),
            "restarts": rng.randint(1, 4), "iters": 20}


# ------------------------------------------------------------------ inputs


def _gen(seed, salt=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + salt)
    return g


def _mixture(n, d, comps, seed, salt=0):
    """(points float32 [n, d], component int64 [n])."""
    g = _gen(seed, salt)
    means = torch.randn(comps, d, generator=g, device="cuda")
    comp = torch.randint(comps, (n,), generator=g, device="cuda")
    return means[comp] + 0.25 * torch.randn(n, d, generator=g, device="cuda"), comp


def _sparse01(n, d, seed):
    """[0, 1]-valued points with 80% of the entries zero: ten noisy means, clipped."""
    g = _gen(seed)
    means = torch.rand(10, d, generator=g, device="cuda")
    comp = torch.randint(10, (n,), generator=g, device="cuda")
    x = (means[comp] + 0.1 * torch.randn(n, d, generator=g, device="cuda")).clamp_(0, 1)
    return x * (torch.rand(n, d, generator=g, device="cuda") >= 0.8)


def _labels(comp, k, seed, part):
    """The components with `part` of them redrawn uniformly, int32."""
    g = _gen(seed, 7)
    n = comp.shape[0]
    other = torch.randint(k, (n,), generator=g, device="cuda")
    return torch.where(torch.rand(n, generator=g, device="cuda") < part, other, comp).to(torch.int32)


def _kernel_args(kernel, d):
    if kernel == "gauss":
        return dict(kernel=kkm.GAUSS, gamma=1.0 / d)
    if kernel == "poly":
        return dict(kernel=kkm.POLY, gamma=1.0, coef0=1.0, degree=2)
    return dict(kernel=kkm.LINEAR)


def _kappa(X, Y, kernel, d):
    """Kernel values of the rows of X against those of Y, in their precision."""
    B = X @ Y.T
    if kernel == "linear":
        return B
    if kernel == "poly":
        return (B + 1.0).square_()
    B.mul_(-2.0).add_((X * X).sum(1)[:, None]).add_((Y * Y).sum(1)[None, :]).clamp_(min=0.0)
    return B.mul_(-1.0 / d).exp_()


def _step_points(case, seed):
    return _mixture(case["n"], 32, case["k"], seed)


def _strip(X, s):
    """Rows of strip s of the Gaussian K over the columns from the strip's first on, float32."""
    a = s * W
    rows = X[a:a + W]
    B = _kappa(rows, X[a:], "gauss", 32)
    r = rows.shape[0]
    D = torch.triu(B[:, :r], 1)
    B[:, :r] = D + D.T
    B[:, :r].fill_diagonal_(1.0)
    return B


def _store(case):
    return torch.bfloat16 if case["store"] == "bf16" else torch.float32


def prepare(case, seed):
    what = case["what"]
    s = {"what": what, "case": case}
    if what == "fit":
        s["X"], comp = _mixture(case["n"], case["d"], case["k"], seed)
        s["labels0"] = _labels(comp, case["k"], seed, 0.5)
    elif what == "step":
        n, k = case["n"], case["k"]
        X, comp = _step_points(case, seed)
        ns = -(-n // W)
        if case["layout"] == "packed":
            K = torch.zeros(kkm.packed_elements(n, PREC[case["store"]]), dtype=_store(case), device="cuda")
            at = 0
            for t in range(ns):
                B = _strip(X, t)
                wide = (ns - t) * W
                K[at:at + B.shape[0] * wide].view(B.shape[0], wide)[:, :B.shape[1]] = B
                at += B.shape[0] * wide
            s["ws"] = torch.empty(kkm.packed_workspace_bytes(n, k, PREC[case["store"]]), dtype=torch.uint8, device="cuda")
        else:
            K = kkm.alloc_kernel_matrix(n, PREC[case["store"]])
            for t in range(ns):
                B = _strip(X, t)
                K[t * W:t * W + B.shape[0], t * W:] = B
                K[t * W:, t * W:t * W + B.shape[0]] = B.T
            s["ws"] = torch.empty(kkm.iterate_workspace_bytes(n, k), dtype=torch.uint8, device="cuda")
        s["K"], s["diag"] = K, torch.ones(n, device="cuda")
        s["labels"] = _labels(comp, k, seed, 0.3)
        s["out"] = _step_outputs(n, k)
    elif what == "gram":
        n, d = case["n"], case["d"]
        s["X"] = _sparse01(n, d, seed) if case["kernel"] == "poly" else _mixture(n, d, 64, seed)[0]
        s["args"] = dict(_kernel_args(case["kernel"], d), gram_prec=PREC[case["prec"]], k_store=PREC[case["store"]])
        if case["layout"] == "packed":
            # columns past n stay as they are here: the product writes K's own entries
            s["K"] = torch.zeros(kkm.packed_elements(n, PREC[case["store"]]), dtype=_store(case), device="cuda")
        else:
            s["K"] = kkm.alloc_kernel_matrix(n, PREC[case["store"]])
        s["diag"] = torch.empty(n, device="cuda")
        s["ws"] = torch.empty(max(kkm.gram_workspace_bytes(n, d, PREC[case["prec"]]), 1), dtype=torch.uint8, device="cuda")
    elif what == "matfree":
        n, d, k = case["n"], case["d"], case["k"]
        s["X"], comp = _mixture(n, d, k, seed)
        s["labels"] = _labels(comp, k, seed, 0.3)
        s["args"] = dict(_kernel_args(case["kernel"], d), gram_prec=PREC[case["prec"]])
        s["ws"] = torch.empty(kkm.matfree_workspace_bytes(n, d, k, PREC[case["prec"]]), dtype=torch.uint8, device="cuda")
        s["out"] = _step_outputs(n, k)
    elif what == "batched":
        s["problems"], s["labels0"] = _batch(case, seed)
        s["ws"] = torch.empty(kkm.kkm_fit_batched_workspace_bytes(s["problems"], PREC[case["prec"]], PREC[case["store"]]),
                              dtype=torch.uint8, device="cuda")
    elif what == "train":
        d = case["d"]
        s["X"] = _mixture(case["B"] * case["steps"], d, 32, seed)[0]
        s["params"] = _network(d, seed)
        s["m"], s["v"] = torch.zeros_like(s["params"]), torch.zeros_like(s["params"])
    else:
        s["X"] = _mixture(case["n"], case["d"], case["k"], seed)[0]
        s["params"] = _network(case["d"], seed)
        s["uniforms"] = np.random.RandomState(seed % (1 << 31)).random_sample((case["restarts"], case["k"]))
    return s


def _step_outputs(n, k):
    return dict(labels_out=torch.empty(n, dtype=torch.int32, device="cuda"),
                counts_out=torch.empty(k, dtype=torch.int32, device="cuda"),
                n_changed=torch.empty(1, dtype=torch.int64, device="cuda"),
                J_in=torch.empty(1, dtype=torch.float64, device="cuda"),
                D_out=torch.empty((n, k), device="cuda"), ctilde_out=torch.empty(k, device="cuda"))


def _sizes(case, seed):
    """(n, d, k) of each problem of a batch: n spread over its range, d and k as the batched workload has them."""
    r = np.random.RandomState((case["count"] * 131 + case["nmax"]) % (1 << 31))
    return [(int(r.randint(case["nmin"], case["nmax"] + 1)), int(r.choice([32, 64, 128, 256])), int(r.randint(2, 65)))
            for _ in range(case["count"])]


def _batch(case, seed):
    problems, labels = [], []
    for b, (n, d, k) in enumerate(_sizes(case, seed)):
        X, comp = _mixture(n, d, k, seed, 100 + b)
        problems.append(dict(X=X, k=k, kernel=kkm.GAUSS, gamma=1.0 / d))
        labels.append(_labels(comp, k, seed * 64 + b, 0.5))
    return problems, torch.cat(labels)


def _network(d, seed, h1=512, h2=512, out=256):
    g, parts = _gen(seed, 11), []
    for rows, cols in ((h1, d), (h2, h1), (out, h2)):
        parts.append((2 * torch.rand(rows * cols, generator=g, device="cuda") - 1) / math.sqrt(cols))
        parts.append(torch.zeros(rows, device="cuda"))
    return torch.cat(parts)


# --------------------------------------------------------------------- run


def run(s):
    what, c = s["what"], s["case"]
    if what == "fit":
        r = kkm.kkm_fit_ex(s["X"], c["k"], s["labels0"], kernel=kkm.GAUSS, gamma=1.0 / c["d"], max_iter=c["iters"],
                           check_convergence=False)
        return r["labels"], r["iters"], r["changed_trace"], np.float32(r["objective"])
    if what == "step":
        f = kkm.kkm_iterate_packed if c["layout"] == "packed" else kkm.kkm_iterate
        r = f(s["K"], s["diag"], s["labels"], c["k"], ws=s["ws"], **s["out"])
        return r[0], r[1], r[2], r[4], r[5]
    if what == "gram":
        f = kkm.kkm_gram_packed if c["layout"] == "packed" else kkm.kkm_gram
        return f(s["X"], K=s["K"], diagK=s["diag"], ws=s["ws"], **s["args"])
    if what == "matfree":
        r = kkm.kkm_iterate_matfree(s["X"], s["labels"], c["k"], ws=s["ws"], **s["args"], **s["out"])
        return r[0], r[1], r[2], r[4], r[5]
    if what == "batched":
        r = kkm.kkm_fit_batched(s["problems"], s["labels0"], PREC[c["prec"]], PREC[c["store"]], max_iter=c["iters"], ws=s["ws"])
        return r["labels"], r["iters"], r["objective"].astype(np.float32)
    if what == "train":
        kkm.kkm_mlp_train_fresh(s["params"], s["m"], s["v"], s["X"], c["B"], gamma=1.0 / c["d"])
        return s["params"], s["m"], s["v"]
    r = kkm.kkm_warm_start(s["params"], s["X"], c["k"], s["uniforms"], max_iter=c["iters"])
    return r["labels"], r["cheap_iters"], r["best"], np.float32(r["objective"])


# -------------------------------------------------------------------- work


def _packed_entries(n):
    ns = -(-n // W)
    return sum(min(W, n - t * W) * (ns - t) * W for t in range(ns))


def work(case):
    what = case["what"]
    size = 2 if case.get("store") == "bf16" else 4
    if what == "fit":
        n, d, k, it = case["n"], case["d"], case["k"], case["iters"]
        # K once, then read once by each iteration and by the final objective
        return {"bytes": 4 * n * (d + n + n * (it + 1)), "flops": n * (n + 1) * d + 2 * n * n * (it + 1)}
    if what == "step":
        n, k = case["n"], case["k"]
        entries = _packed_entries(n) if case["layout"] == "packed" else n * n
        return {"bytes": entries * size + 4 * n * k + 12 * n, "flops": n * n}
    if what == "gram":
        n, d = case["n"], case["d"]
        entries = _packed_entries(n) if case["layout"] == "packed" else n * n
        return {"bytes": 4 * n * d + entries * size, "flops": n * (n + 1) * d}
    if what == "matfree":
        n, d, k = case["n"], case["d"], case["k"]
        return {"bytes": 4 * n * (d + k) + 12 * n, "flops": n * (n + 1) * d + n * n}
    if what == "batched":
        # K once and at least two steps (one that changes labels, one that changes none)
        nn = [(n, d) for n, d, _ in _sizes(case, 0)]
        return {"bytes": sum(4 * n * d + 3 * size * n * n for n, d in nn), "flops": sum(n * (n + 1) * d for n, d in nn)}
    if what == "train":
        d, B, steps = case["d"], case["B"], case["steps"]
        weights = 512 * d + 512 * 512 + 256 * 512
        return {"bytes": steps * (28 * weights + 4 * B * d), "flops": steps * (6 * B * weights + 6 * B * B * 256 + B * B * d)}
    n, d, k = case["n"], case["d"], case["k"]
    weights = 512 * d + 512 * 512 + 256 * 512
    rounds = case["restarts"] * (k + 2)  # every seed and at least two Lloyd steps read the features
    return {"bytes": 4 * n * d + 4 * n * 256 * rounds, "flops": 2 * n * weights + case["restarts"] * 4 * n * 256 * k}


# ------------------------------------------------------------------- exact


def _distances(rows_of, n, k, labels, diag):
    """(D [n, k], centroid norms [k]) in float64; rows_of(a, b) gives rows a..b of K."""
    lab = labels.long()
    one = torch.zeros(n, k, dtype=torch.float64, device="cuda")
    one[torch.arange(n, device="cuda"), lab] = 1.0
    cnt = one.sum(0)
    E = torch.cat([rows_of(a, min(a + W, n)) @ one for a in range(0, n, W)]) / cnt
    own = E[torch.arange(n, device="cuda"), lab]
    norms = torch.zeros(k, dtype=torch.float64, device="cuda").index_add_(0, lab, own) / cnt
    empty = cnt == 0
    norms[empty] = 0.0
    D = diag.double()[:, None] - 2.0 * E + norms
    D[:, empty] = math.inf
    return D, norms


def _fit(X, k, labels, d, iters, converge):
    """(iterations, objective of the final labels) of a run in float64."""
    X = X.double()
    n = X.shape[0]
    K = _kappa(X, X, "gauss", d).fill_diagonal_(1.0)
    one = torch.ones(n, device="cuda")
    t = 0
    while t < iters:
        D, _ = _distances(lambda a, b: K[a:b], n, k, labels, one)
        new = D.argmin(1)
        t += 1
        same = bool((new == labels).all())
        labels = new
        if converge and same:
            break
    D, _ = _distances(lambda a, b: K[a:b], n, k, labels, one)
    return t, float(D[torch.arange(n, device="cuda"), labels.long()].sum())


def exact(case, seed):
    what = case["what"]
    if what == "fit":
        s = prepare(case, seed)
        _, J = _fit(s["X"], case["k"], s["labels0"], case["d"], case["iters"], False)
        return None, None, None, J
    if what == "step":
        n, k = case["n"], case["k"]
        X, comp = _step_points(case, seed)
        lab = _labels(comp, k, seed, 0.3)
        lo = torch.zeros(n, k, dtype=torch.float64, device="cuda")
        one = torch.nn.functional.one_hot(lab.long(), k).double()
        for t in range(-(-n // W)):
            a = t * W
            B = _strip(X, t).to(_store(case)).double()
            r = B.shape[0]
            lo[a:a + r] += B @ one[a:]
            lo[a + r:] += B[:, r:].T @ one[a:a + r]
        # the sums are at hand: rows_of's product with the indicators is replaced by them
        cnt = one.sum(0)
        E = lo / cnt
        own = E[torch.arange(n, device="cuda"), lab.long()]
        norms = torch.zeros(k, dtype=torch.float64, device="cuda").index_add_(0, lab.long(), own) / cnt
        norms[cnt == 0] = 0.0
        D = 1.0 - 2.0 * E + norms
        D[:, cnt == 0] = math.inf
        return None, None, None, D, norms
    if what == "gram":
        s = prepare(case, seed)
        n, d = case["n"], case["d"]
        X = s["X"].double()
        del s["K"]
        ns = -(-n // W)
        if case["layout"] == "packed":
            K = torch.zeros(kkm.packed_elements(n, PREC[case["store"]]), dtype=torch.float64, device="cuda")
            at = 0
            for t in range(ns):
                B = _kappa(X[t * W:(t + 1) * W], X[t * W:], case["kernel"], d)
                wide = (ns - t) * W
                K[at:at + B.shape[0] * wide].view(B.shape[0], wide)[:, :B.shape[1]] = B
                at += B.shape[0] * wide
        else:
            K = torch.empty(n, n, dtype=torch.float64, device="cuda")
            for t in range(ns):
                K[t * W:(t + 1) * W] = _kappa(X[t * W:(t + 1) * W], X, case["kernel"], d)
        q = (X * X).sum(1)
        return K, torch.ones_like(q) if case["kernel"] == "gauss" else (q + 1.0) ** 2 if case["kernel"] == "poly" else q
    if what == "matfree":
        s = prepare(case, seed)
        X, d = s["X"].double(), case["d"]
        q = (X * X).sum(1)
        diag = torch.ones_like(q) if case["kernel"] == "gauss" else (q + 1.0) ** 2
        D, norms = _distances(lambda a, b: _kappa(X[a:b], X, case["kernel"], d), case["n"], case["k"], s["labels"], diag)
        return None, None, None, D, norms
    if what == "batched":
        problems, labels0 = _batch(case, seed)
        J, at = [], 0
        for p in problems:
            n, d = p["X"].shape
            J.append(_fit(p["X"], p["k"], labels0[at:at + n], d, case["iters"], True)[1])
            at += n
        return None, None, np.array(J)
    return None  # bfloat16 roundings inside the network decide its last digits
