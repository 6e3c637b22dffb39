"""Performance cases: what users of the tree-ensemble scorer have it do, over the range they do it in.

Models and documents are synthetic and seeded, shaped like the repository's workloads: random
unbalanced trees (n_leaves - 1 splits of a leaf chosen uniformly) or complete trees, thresholds
drawn where the feature values lie, documents with a share of exact zeros. A pass is one call of
the public binding on documents that are already on the GPU, with a model packed beforehand.

  listed()             the cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  the packed model and the documents of a case
  run(state)           one pass
  work(case)           bytes and comparisons a pass cannot do without
  tolerance(case)      how far outputs of another correct implementation may lie
  exact(case, seed)    the outputs in 64 bits, by plain torch
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1212_2287_amd as te

# One case: the call, the model's shape, the documents. `leaves` is the largest tree, trees are
# uniform on [min_leaves, leaves]; `depth` caps random trees (0: no cap; log2(leaves) makes them
# complete). `thresholds`: "sample" = distributed like the feature's values (zeros included),
# "nonzero" = like its nonzero values.
_BASE = {"call": "predict", "trees": 1000, "leaves": 32, "min_leaves": 32, "depth": 16, "features": 136,
         "docs": 100_000, "zeros": 0.3, "values": "lognormal", "thresholds": "sample", "sigma": 0.1,
         "outputs": 1, "bags": 1, "strict": False, "k": 0}


def _case(**changes) -> dict:
    return {**_BASE, **changes}


def listed() -> list:
    return [
        # a small early-stage filter over one shard's candidates: bound by launch and call overhead
        _case(name="tiny_10x8", trees=10, leaves=8, min_leaves=8, depth=0, docs=1_000, zeros=0.0,
              values="uniform", sigma=1.0),
        # online serving: one query's 100 candidates through the ranking model
        _case(name="serve_100docs", docs=100),
        # a validation fold scored by a model of mixed tree sizes over 46 features (LETOR's width),
        # with the strict tie rule; an odd batch that fills a fraction of the GPU
        _case(name="letor_300_f46", trees=300, leaves=200, min_leaves=2, depth=0, features=46, docs=4_097,
              zeros=0.1, values="uniform", strict=True),
        # a service's micro-batch of queries: score and keep each query's 20 best
        _case(name="rerank_20k_top20", call="predict_topk", docs=20_000, k=20),
        # the learning-to-rank test set (MSLR's width), the repository's main workload
        _case(name="rank_1kx32", docs=100_000),
        # wide documents, sparse features
        _case(name="wide_1kx64_f700", leaves=64, min_leaves=64, depth=20, features=700, docs=50_000, zeros=0.6,
              values="uniform", thresholds="nonzero"),
        # long boosting run of shallow complete trees over a large collection
        _case(name="shallow_20kx8_1M", trees=20_000, leaves=8, min_leaves=8, depth=3, docs=1_000_000, zeros=0.0,
              values="uniform", sigma=0.01),
        # the largest model and collection: 5,000 trees of 256 leaves over 700 features
        _case(name="large_5kx256_f700_1M", trees=5_000, leaves=256, min_leaves=256, depth=24, features=700,
              docs=1_000_000, zeros=0.5, sigma=0.01),
        # leaf ids as features of a downstream linear model (or for a parity check)
        _case(name="leaf_ids_30k", call="leaves", docs=30_011),
        # multi-output regression, two bagged ensembles averaged
        _case(name="multi_8_outputs", outputs=8, bags=2, docs=50_000),
        # which features a prediction reads (the access study of the paper's Section 6): about 95%
        # of them per document, as on the paper's MSLR models
        _case(name="trace_100k", call="usage", trees=100),
        # a random forest of deep trees, each larger than an LDS tile
        _case(name="forest_32x4096", trees=32, leaves=4_096, min_leaves=4_096, depth=0, docs=20_000,
              sigma=1.0, bags=32),
    ]


def _log_int(rng, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng) -> dict:
    kind = rng.choice(["serve", "rank", "rank", "wide", "shallow", "deep", "topk", "leaves", "multi", "usage", "forest"])
    c = _case(zeros=rng.choice([0.0, 0.3, 0.5]), values=rng.choice(["uniform", "lognormal"]),
              strict=rng.random() < 0.25, features=_log_int(rng, 20, 160), depth=0)
    budget = 2.0e10  # comparisons of a pass at most
    if kind == "serve":
        c.update(trees=_log_int(rng, 10, 2_000), leaves=_log_int(rng, 4, 64), docs=_log_int(rng, 1, 2_000))
    elif kind == "rank":
        c.update(trees=_log_int(rng, 100, 5_000), leaves=_log_int(rng, 8, 128), docs=_log_int(rng, 2_000, 1_000_000))
    elif kind == "wide":
        c.update(trees=_log_int(rng, 100, 2_000), leaves=_log_int(rng, 8, 128), features=_log_int(rng, 160, 1_000),
                 docs=_log_int(rng, 1_000, 200_000), thresholds="nonzero")
    elif kind == "shallow":
        depth = rng.randint(2, 6)
        c.update(trees=_log_int(rng, 200, 20_000), leaves=1 << depth, depth=depth, docs=_log_int(rng, 1_000, 1_000_000))
    elif kind == "deep":
        c.update(trees=_log_int(rng, 50, 5_000), leaves=_log_int(rng, 128, 512), features=_log_int(rng, 46, 760),
                 docs=_log_int(rng, 1_000, 300_000))
    elif kind == "topk":
        c.update(call="predict_topk", trees=_log_int(rng, 100, 1_000), leaves=_log_int(rng, 8, 64),
                 docs=_log_int(rng, 100, 200_000), k=rng.choice([5, 10, 20, 64]))
    elif kind == "leaves":
        c.update(call="leaves", trees=_log_int(rng, 10, 2_000), leaves=_log_int(rng, 8, 64), docs=_log_int(rng, 100, 40_000))
    elif kind == "multi":
        c.update(trees=_log_int(rng, 100, 1_000), leaves=_log_int(rng, 8, 64), docs=_log_int(rng, 500, 60_000),
                 outputs=rng.randint(2, 12), bags=rng.randint(1, 4))
    elif kind == "usage":
        c.update(call="usage", trees=_log_int(rng, 10, 1_000), leaves=_log_int(rng, 8, 64), docs=_log_int(rng, 500, 100_000),
                 features=_log_int(rng, 20, 500))
    else:
        c.update(trees=_log_int(rng, 8, 48), leaves=_log_int(rng, 3_100, 5_000), docs=_log_int(rng, 500, 30_000), sigma=1.0)
    # half of the random models mix tree sizes
    mixed = kind not in ("shallow", "forest") and rng.random() < 0.5
    c["min_leaves"] = 2 if mixed else c["leaves"]
    most = budget / (c["trees"] * _path(c))
    c["docs"] = int(max(1, min(c["docs"], most, 7.0e8 / c["features"])))
    return c


def _path(case: dict) -> float:
    """Mean comparisons of a walk: each split of the growing tree meets the document's leaf with
    probability 1 / (leaves so far), so H(leaves - 1); complete trees their depth."""
    if case["depth"] and 1 << case["depth"] == case["leaves"]:
        return float(case["depth"])
    n = (case["leaves"] + case["min_leaves"]) // 2
    return max(1.0, math.log(n) + 0.577)


# ----------------------------------------------------------------------------------------------
# inputs
# ----------------------------------------------------------------------------------------------
def _model(case: dict, seed: int) -> dict:
    """Flat creation-order arrays of the model (all trees grown together, split by split)."""
    rng = np.random.default_rng([seed, 1])
    T, L, F = case["trees"], case["leaves"], case["features"]
    n_leaves = np.full(T, L) if case["min_leaves"] == L else rng.integers(case["min_leaves"], L + 1, T)
    n_leaves[0] = L
    N = 2 * L - 1
    feature = np.full((T, N), -1, np.int32)
    left = np.full((T, N), -1, np.int32)
    depth = np.zeros((T, N), np.int32)
    open_, count = np.zeros((T, L), np.int32), np.ones(T, np.int64)  # leaves that may be split
    cap = case["depth"] or N
    rows = np.arange(T)
    for s in range(L - 1):
        r = rows if case["min_leaves"] == L else np.nonzero(n_leaves > s + 1)[0]
        at = (rng.random(r.size) * count[r]).astype(np.int64)
        node = open_[r, at]
        count[r] -= 1
        open_[r, at] = open_[r, count[r]]
        feature[r, node] = rng.integers(0, F, r.size)
        left[r, node] = 2 * s + 1
        d = depth[r, node] + 1
        depth[r, 2 * s + 1] = depth[r, 2 * s + 2] = d
        more = r[d < cap]
        open_[more, count[more]] = 2 * s + 1
        open_[more, count[more] + 1] = 2 * s + 2
        count[more] += 2
    keep = np.arange(N)[None, :] < (2 * n_leaves - 1)[:, None]
    feature, left = feature[keep], left[keep]
    inner = feature >= 0
    n, k = feature.size, int(inner.sum())
    thr = np.zeros(n, np.float32)
    t = rng.random(k, np.float32) if case["values"] == "uniform" else np.exp(rng.standard_normal(k, np.float32))
    if case["thresholds"] == "sample":
        t[rng.random(k, np.float32) < case["zeros"]] = 0.0
    thr[inner] = t
    shape = (n,) if case["outputs"] == 1 else (n, case["outputs"])
    value = rng.standard_normal(shape, np.float32) * np.float32(case["sigma"])
    value[inner] = 0.0
    offsets = np.concatenate([[0], np.cumsum(2 * n_leaves - 1)]).astype(np.int64)
    return {"offsets": offsets, "feature": feature, "threshold": thr, "left": left,
            "right": np.where(inner, left + 1, -1).astype(np.int32), "value": value}


def _docs(case: dict, seed: int) -> torch.Tensor:
    g = torch.Generator(device="cuda").manual_seed(2 * seed + 1)
    n, F = case["docs"], case["features"]
    X = torch.empty((n, F), dtype=torch.float32, device="cuda")
    step = max(1, 1 << 27) // F
    for a in range(0, n, step):
        x = X[a:a + step]
        x.uniform_(generator=g) if case["values"] == "uniform" else x.normal_(generator=g).exp_()
        if case["zeros"]:
            x.masked_fill_(torch.rand(x.shape, generator=g, device="cuda") < case["zeros"], 0.0)
    return X


def _groups(case: dict, seed: int) -> np.ndarray:
    """Offsets of query groups of about 20 to 200 documents, 110 on average."""
    sizes = np.random.default_rng([seed, 2]).integers(20, 201, max(1, case["docs"] // 110))
    ends = np.cumsum(sizes) * (case["docs"] / sizes.sum())
    return np.concatenate([[0], np.rint(ends)]).astype(np.int64)


def prepare(case: dict, seed: int) -> dict:
    m = _model(case, seed)
    flags = te.TREE_ENS_RIGHT_IF_GT if case["strict"] else te.TREE_ENS_RIGHT_IF_GE
    model = te.TreeEnsemble.from_arrays(m["offsets"], m["feature"], m["threshold"], m["left"], m["right"], m["value"],
                                        flags, case["outputs"], case["bags"])
    state = {"call": case["call"], "model": model, "X": _docs(case, seed), "k": case["k"]}
    if case["call"] == "predict_topk":
        state["groups"] = torch.from_numpy(_groups(case, seed)).cuda()
    return state


def run(state: dict):
    model, X = state["model"], state["X"]
    if state["call"] == "predict":
        return model.predict(X)
    if state["call"] == "predict_topk":
        return model.predict_topk(X, state["groups"], state["k"])
    if state["call"] == "leaves":
        return model.predict_leaves(X)
    return model.feature_usage(X)


# ----------------------------------------------------------------------------------------------
# what a pass needs, and how close its outputs have to be
# ----------------------------------------------------------------------------------------------
def work(case: dict) -> dict:
    n, T = case["docs"], case["trees"]
    nodes = T * ((case["leaves"] + case["min_leaves"]) - 1)
    out = {"predict": 4 * n * case["outputs"], "predict_topk": 4 * n + max(1, n // 110) * (8 + 8 * case["k"]),
           "leaves": 4 * n * T, "usage": n * (4 + 4 * ((case["features"] + 31) // 32))}[case["call"]]
    # a node: a threshold, a feature id and a link (8 bytes); a leaf row: n_outputs floats
    model = nodes * 8 + (nodes / 2 * 4 * case["outputs"] if case["outputs"] > 1 else 0)
    sums = 0 if case["call"] in ("leaves", "usage") else case["outputs"]
    return {"bytes": float(4 * n * case["features"] + out + model), "flops": float(n * T * (_path(case) + sums))}


def tolerance(case: dict):
    # Leaf ids and feature sets are whole numbers. Scores are double sums rounded once to float:
    # the rounding alone is 2.5e-8 to 3e-8 of the result (2-norm), whatever the order of the sum.
    if case["call"] in ("leaves", "usage"):
        return "exact"
    tol = {"rel": 1.2e-7}
    if case["call"] == "predict_topk":
        tol["differ"] = 1e-3  # documents whose scores are one rounding apart
    return tol


def exact(case: dict, seed: int):
    """The outputs in 64 bits: every tree walked by plain indexing, leaf values summed in double."""
    n, T, O = case["docs"], case["trees"], case["outputs"]
    if n * T * _path(case) > 2.5e10:
        return None
    m = _model(case, seed)
    X = _docs(case, seed)
    dev = {k: torch.from_numpy(v).cuda() for k, v in m.items()}
    off, fe, th, le = dev["offsets"][:-1], dev["feature"].long(), dev["threshold"], dev["left"].long()
    val = dev["value"].double().reshape(-1, O)
    words = (case["features"] + 31) // 32
    scores = torch.empty((n, O), dtype=torch.float64, device="cuda")
    leaf = torch.empty((n, T) if case["call"] == "leaves" else (0, T), dtype=torch.int32, device="cuda")
    masks = torch.zeros((n, words) if case["call"] == "usage" else (0, words), dtype=torch.int32, device="cuda")
    counts = torch.zeros(n if case["call"] == "usage" else 0, dtype=torch.int32, device="cuda")
    step = max(1, 12_000_000 // (T * max(1, O // 2)))
    for a in range(0, n, step):
        x = X[a:a + step]
        at = off.expand(x.shape[0], T)
        seen = torch.zeros((x.shape[0], words * 32 + 1), dtype=torch.bool, device="cuda") if masks.numel() else None
        while True:
            f = fe[at]
            inner = f >= 0
            if not bool(inner.any()):
                break
            if seen is not None:  # leaves mark the spare last column
                seen.scatter_(1, torch.where(inner, f, words * 32), True)
            v, t = x.gather(1, f.clamp_min(0)), th[at]
            right = v > t if case["strict"] else v >= t
            at = torch.where(inner, off + le[at] + right, at)
        if case["call"] == "leaves":
            leaf[a:a + step] = (at - off).int()
        elif seen is not None:
            bits = seen[:, :words * 32].view(-1, words, 32).long()
            word = (bits << torch.arange(32, device="cuda")).sum(2)
            masks[a:a + step] = torch.where(word >= 1 << 31, word - (1 << 32), word).int()
            counts[a:a + step] = bits.sum((1, 2)).int()
        else:
            scores[a:a + step] = val[at].sum(1) / case["bags"]
    if case["call"] == "leaves":
        return leaf
    if case["call"] == "usage":
        return counts, masks
    scores = scores[:, 0] if O == 1 else scores
    if case["call"] == "predict":
        return scores
    groups, k = _groups(case, seed), case["k"]
    idx = torch.full((groups.size - 1, k), -1, dtype=torch.int32)
    top = torch.full((groups.size - 1, k), math.nan, dtype=torch.float64)
    host = scores.cpu()
    for g, (a, b) in enumerate(zip(groups[:-1], groups[1:])):
        s, order = torch.sort(host[a:b], descending=True, stable=True)
        c = min(k, int(b - a))
        idx[g, :c] = (order[:c] + int(a)).int()
        top[g, :c] = s[:c]
    return scores, idx, top
