"""The work that a user of this library has it do, as cases that can be timed and compared.

A case is a dict of plain values: the forest (``shape``, ``trees``, ``depth``, ``features``,
``classes``, ``vector`` leaves, ``mean``, ``link``), the rows (``rows``, ``x``) and the call
(``call``, ``pre`` for a fused scaler).  Forests and rows are synthetic and drawn from the seed:

* ``shape`` "perfect": every leaf at ``depth`` (depth-wise boosting with full trees); "ragged":
  every node above ``depth`` splits with probability 0.85; "grown": trees grown until each leaf
  holds one of ``samples`` training rows, as random forests without a depth limit are.
* ``x`` "normal": N(0, 1); "sparse": U[0, 1) with 80% zeros (pixels, counts, one-hot text).
* ``call`` "predict", "labels", "leaves" (leaf ids), "binned" (bin the rows, then predict from
  the bins) or "csr" (predict from compressed sparse rows).
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2405_12491_amd as B

SPLIT = 0.85
KEEP = 0.2
LINKS = {"none": B.BRIDGER_XFORM_IDENTITY, "sigmoid": B.BRIDGER_XFORM_SIGMOID,
         "softmax": B.BRIDGER_XFORM_SOFTMAX}
PRES = {"none": B.BRIDGER_PRE_NONE, "minmax": B.BRIDGER_PRE_MINMAX,
        "standard": B.BRIDGER_PRE_CENTER_SCALE, "binarize": B.BRIDGER_PRE_BINARIZE,
        "normalize": B.BRIDGER_PRE_NORMALIZE}

BASE = dict(shape="perfect", trees=100, depth=6, samples=0, features=28, classes=1, vector=False,
            mean=False, link="none", rows=1000, x="normal", call="predict", pre="none")


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one decision tree on a small table: latency of a call
        _case("one_tree_10k", trees=1, depth=3, rows=10_000),
        # a serving batch of a binary boosted classifier: too few rows to fill the chip
        _case("gbdt_serving_1k", trees=500, link="sigmoid", rows=1_000),
        # the same model over a whole table, the benchmark's workload
        _case("gbdt_1m", trees=500, link="sigmoid", rows=1_000_000),
        # leaf ids of a boosted model as features of a linear model (leaf embedding)
        _case("gbdt_leaves_200k", trees=500, rows=200_000, call="leaves"),
        # quantized rows: a random forest's bins, then the prediction from them
        _case("rf_binned_1m", trees=100, depth=8, mean=True, rows=1_000_000, call="binned"),
        # ten classes on wide rows (784 pixels), dense ...
        _case("mc_gbdt_wide_100k", trees=1000, depth=8, features=784, classes=10, link="softmax",
              rows=100_000, x="sparse"),
        # ... and the same rows as they come from a sparse pipeline
        _case("mc_gbdt_csr_50k", trees=1000, depth=8, features=784, classes=10, link="softmax",
              rows=50_000, x="sparse", call="csr"),
        # a scaler and a multiclass model, labels out, on the 51,630 x 90 shape of the paper's
        # tabular set (rows not 16-byte aligned)
        _case("scaled_labels_52k", trees=300, depth=6, features=90, classes=5, link="softmax",
              rows=51_630, call="labels", pre="standard"),
        # a large ragged forest over a large table
        _case("ragged_wide_4m", shape="ragged", trees=1000, depth=12, features=256,
              rows=4_000_000),
        # a random-forest classifier: class probabilities in the leaves, ragged trees
        _case("rf_classifier_300k", shape="ragged", trees=100, depth=12, classes=7, vector=True,
              mean=True, rows=300_000),
        # a small odd batch of a ragged regression forest
        _case("ragged_serving_3k", shape="ragged", trees=100, depth=12, mean=True, rows=3_001),
        # fully grown trees of tens of thousands of nodes
        _case("grown_52k", shape="grown", trees=64, depth=0, samples=20_000, features=90, mean=True,
              rows=51_630),
    ]


def _loguniform(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    shape = rng.choice(["perfect", "perfect", "perfect", "ragged", "ragged", "ragged", "grown"])
    wide = rng.random() < 0.3
    c = _case(shape=shape, features=_loguniform(rng, 200, 900) if wide else _loguniform(rng, 6, 120),
              x=rng.choice(["normal", "sparse"] if wide else ["normal", "normal", "sparse"]))
    if shape == "grown":
        c.update(depth=0, samples=_loguniform(rng, 17_000, 30_000), trees=_loguniform(rng, 10, 60))
    elif shape == "ragged":
        c.update(depth=rng.randint(5, 13), trees=_loguniform(rng, 20, 600))
    else:
        c.update(depth=rng.randint(3, 9), trees=_loguniform(rng, 1, 1000))
    if rng.random() < 0.4 and c["trees"] >= 20:
        c["classes"] = rng.randint(2, 12)
        c["vector"] = rng.random() < 0.5
    c["mean"] = c["vector"] or rng.random() < 0.3
    if c["classes"] > 1:
        c["link"] = "none" if c["vector"] else rng.choice(["softmax", "softmax", "none"])
    else:
        c["link"] = rng.choice(["none", "sigmoid"])
    calls = ["predict", "predict", "predict", "leaves"]
    if shape != "grown":
        calls += ["binned"] + (["csr"] if c["x"] == "sparse" else [])
    if (c["classes"] > 1 and not c["vector"]) or c["link"] == "sigmoid":
        calls += ["labels"]
    c["call"] = rng.choice(calls)
    c["pre"] = rng.choice(["none"] * 5 + ["minmax", "standard", "normalize", "binarize"])
    # rows: from a handful to a table, no more work than the listed cases
    visits = c["trees"] * (_path(c) + (c["classes"] if c["vector"] else 1))
    most = min(1_000_000, int(4e9 / visits), int(3e8 / c["features"]))
    if c["call"] == "leaves":
        most = min(most, int(8e7 / c["trees"]))
    if shape == "grown":
        most = min(most, 60_000)
    c["rows"] = _loguniform(rng, min(50, most), most)
    return c


# ------------------------------------------------------------------------------ inputs
def _path(c):
    """Mean number of comparisons of a row in a tree."""
    if c["shape"] == "perfect":
        return float(c["depth"])
    if c["shape"] == "ragged":
        return sum(SPLIT ** (d + 1) for d in range(c["depth"]))
    return 1.25 * math.log2(c["samples"])


def _nodes(c):
    """Nodes of one tree (about)."""
    if c["shape"] == "perfect":
        return 2.0 ** (c["depth"] + 1) - 1
    if c["shape"] == "ragged":
        return 1.0 + sum((2 * SPLIT) ** (d + 1) for d in range(c["depth"]))
    return 2.0 * c["samples"] - 1


def _forest(case, seed):
    """The model's arrays (nodes breadth-first in each tree), as a frontend hands them over."""
    rng = np.random.default_rng([seed, 2])
    T, F, K = case["trees"], case["features"], case["classes"]
    limit = 64 if case["shape"] == "grown" else case["depth"]
    tree = np.arange(T)                      # tree of each node of the level
    count = np.full(T, max(case["samples"], 1))  # training rows of each node ("grown")
    before = np.zeros(T, np.int64)           # nodes of each tree above the level
    levels = []
    for d in range(limit + 1):
        n = len(tree)
        per = np.bincount(tree, minlength=T)
        first = np.concatenate([[0], np.cumsum(per)[:-1]])
        local = before[tree] + np.arange(n) - first[tree]
        share = np.full(n, 0.5)
        if d == limit:
            split = np.zeros(n, bool)
        elif case["shape"] == "grown":
            split = count > 1
            share = rng.uniform(0.15, 0.85, n)
        else:
            split = np.ones(n, bool) if case["shape"] == "perfect" else rng.random(n) < SPLIT
        before = before + per
        kids = tree[split]
        rank = np.arange(len(kids)) - np.concatenate([[0], np.cumsum(np.bincount(kids, minlength=T))[:-1]])[kids]
        left = np.full(n, -1, np.int64)
        left[split] = before[kids] + 2 * rank
        lc = np.clip(np.rint(count[split] * share[split]), 1, np.maximum(count[split] - 1, 1)) \
            if case["shape"] == "grown" else np.ones(len(kids))
        levels.append((tree, local, left, share))
        count = np.stack([lc, count[split] - lc], 1).reshape(-1).astype(np.int64) \
            if case["shape"] == "grown" else np.ones(2 * len(kids), np.int64)
        tree = np.repeat(kids, 2)
        if not len(tree):
            break
    offs = np.concatenate([[0], np.cumsum(before)]).astype(np.int64)
    N = int(offs[-1])
    left = np.full(N, -1, np.int32)
    share = np.full(N, 0.5)
    for t, local, l, s in levels:
        left[offs[t] + local] = l
        share[offs[t] + local] = s
    inner = left >= 0
    right = np.where(inner, left + 1, -1).astype(np.int32)
    feature = np.where(inner, rng.integers(0, F, N), -1).astype(np.int32)
    if case["pre"] == "binarize":
        thr = np.full(N, 0.5, np.float32)
    elif case["shape"] == "grown" and case["x"] == "normal":  # a row goes left with the node's share
        thr = torch.special.ndtri(torch.from_numpy(share)).numpy()
    elif case["x"] == "normal":
        thr = rng.standard_normal(N, dtype=np.float32)
    else:
        thr = np.where(rng.random(N) < KEEP, rng.random(N, dtype=np.float32), 0.0)
    thr = np.asarray(thr, np.float64)
    if case["pre"] == "minmax":
        thr = thr * 0.25 + 0.5
    elif case["pre"] == "normalize":
        thr = thr / math.sqrt(F)
    thr = np.where(inner, thr, 0.0).astype(np.float32)
    if case["vector"]:
        value = rng.random((N, K), dtype=np.float32) ** 4
        value /= value.sum(1, keepdims=True)
    else:
        value = rng.standard_normal(N, dtype=np.float32) * np.float32(1.0 if case["mean"] else 0.1)
    value[inner] = 0.0
    return SimpleNamespace(
        n_features=F, n_classes=K, tree_offsets=offs, feature=feature, threshold=thr, left=left,
        right=right, value=np.ascontiguousarray(value),
        tree_class=None if K == 1 or case["vector"] else (np.arange(T) % K).astype(np.int32),
        aggregate=B.BRIDGER_AGG_MEAN if case["mean"] else B.BRIDGER_AGG_SUM,
        transform=LINKS[case["link"]], base_score=None)


def _rows(case, seed):
    """The row matrix, float32 [rows, features], on the GPU."""
    g = torch.Generator(device="cuda").manual_seed(1_000_003 * (seed % 1_000_003) + 1)
    shape = (case["rows"], case["features"])
    if case["x"] == "normal":
        return torch.randn(shape, generator=g, device="cuda")
    X = torch.rand(shape, generator=g, device="cuda")
    X *= torch.rand(shape, generator=g, device="cuda") < KEEP
    return X


def _scaler(case, seed):
    """Parameters a, b of the fused preprocessing step (float64 [features] or None)."""
    rng = np.random.default_rng([seed, 3])
    F, pre = case["features"], case["pre"]
    if pre == "minmax":
        return rng.uniform(0.2, 0.3, F), rng.uniform(0.4, 0.6, F)
    if pre == "standard":
        return rng.normal(0.0, 0.1, F), rng.uniform(0.8, 1.25, F)
    if pre == "binarize":
        return rng.normal(0.0, 0.3, F) if case["x"] == "normal" else rng.uniform(0.0, 0.5, F), None
    return None, None


def prepare(case, seed):
    forest = B.Forest(_forest(case, seed))
    if case["pre"] != "none":
        forest.set_preprocess(PRES[case["pre"]], *_scaler(case, seed))
    X = _rows(case, seed)
    state = {"forest": forest, "call": case["call"], "rows": case["rows"]}
    if case["call"] == "csr":
        stored = X != 0
        state["indptr"] = torch.zeros(case["rows"] + 1, dtype=torch.int64, device="cuda")
        torch.cumsum(stored.sum(1), 0, out=state["indptr"][1:])
        state["indices"] = stored.nonzero()[:, 1].to(torch.int32)
        state["values"] = X[stored]
    else:
        state["X"] = X
    return state


def run(state):
    f, call = state["forest"], state["call"]
    if call == "csr":
        return f.predict_csr(state["indptr"], state["indices"], state["values"], state["rows"])
    X = state["X"]
    if call == "labels":
        return f.predict_labels(X)
    if call == "leaves":
        return f.predict_leaves(X)
    if call == "binned":
        bins = f.bin(X)
        return {"bins": bins, "scores": f.predict_binned(bins)}
    return f.predict(X)


# -------------------------------------------------------------------- work and tolerance
def work(case):
    """Rows in, results out, the forest once (8 bytes a node: threshold and feature, or a
    leaf's value; a vector leaf's class values), or what the rows' paths visit of it where that
    is less; two operations a comparison and an addition for each value added."""
    n, T, K, F = case["rows"], case["trees"], case["classes"], case["features"]
    adds = K if case["vector"] else 1
    forest = T * _nodes(case) * 6.0 + T * _nodes(case) * 2.0 * adds
    visited = n * T * (_path(case) * 8.0 + 4.0 * adds)
    if case["call"] == "csr":
        rows_in = n * F * KEEP * 8.0 + (n + 1) * 8.0
    else:
        rows_in = n * F * 4.0
    out = n * {"labels": 4.0, "leaves": 4.0 * T}.get(case["call"], 4.0 * K)
    flops = n * T * (2.0 * _path(case) + (0 if case["call"] == "leaves" else adds))
    if case["call"] == "binned":  # the bins are an output too (2 bytes, or 1 with few thresholds)
        per_feature = T * _nodes(case) / 2 / F
        bin_bytes = n * F * (2.0 if per_feature > 300 else 1.0)
        out += bin_bytes
        flops += n * F * math.log2(max(per_feature, 2.0))
    return {"bytes": rows_in + out + min(forest, visited), "flops": flops}


def tolerance(case):
    """Sums are kept in double precision and rounded to float once: another order of the sums
    changes at most the last bit of a value.  Labels, leaf ids and bins are whole numbers."""
    if case["call"] in ("labels", "leaves"):
        return "exact"
    return {"rel": 1.2e-7, "max": 5e-7}


# ---------------------------------------------------------------------------- 64 bits

def _scaled(case, seed, X):
    """The preprocessing as it is defined: each step in 64 bits, rounded to float."""
    pre = case["pre"]
    if pre == "none":
        return X
    if pre == "normalize":
        norm = X.double().square().sum(1, keepdim=True).sqrt()
        return (X.double() / torch.where(norm == 0, torch.ones_like(norm), norm)).float()
    a, b = (None if v is None else torch.from_numpy(np.asarray(v)).to(X.device)
            for v in _scaler(case, seed))
    if pre == "minmax":
        return ((X.double() * a).float().double() + b).float()
    if pre == "standard":
        return ((X.double() - a).float().double() / b).float()
    return (X.double() > a).float()


def exact(case, seed):
    """Scores in 64 bits: every tree walked level by level over all rows."""
    if case["call"] in ("labels", "leaves"):
        return None
    f = _forest(case, seed)
    X = _scaled(case, seed, _rows(case, seed))
    n, K, T = case["rows"], case["classes"], case["trees"]
    dev = X.device
    feature, threshold, left, value = (torch.from_numpy(v).to(dev)
                                       for v in (f.feature, f.threshold, f.left, f.value))
    feature = feature.long()
    acc = torch.zeros((n, K), dtype=torch.float64, device=dev)
    for t in range(T):
        lo, hi = int(f.tree_offsets[t]), int(f.tree_offsets[t + 1])
        feat, thr, lft = feature[lo:hi], threshold[lo:hi], left[lo:hi].long()
        node = torch.zeros(n, dtype=torch.int64, device=dev)
        for _ in range(64 if case["shape"] == "grown" else case["depth"]):
            fn, ln = feat[node], lft[node]
            inner = ln >= 0
            x = X.gather(1, fn.clamp_(min=0).unsqueeze(1)).squeeze(1)
            node = torch.where(inner, ln + ~(x <= thr[node]), node)
        v = value[lo:hi][node].double()
        if case["vector"]:
            acc += v
        else:
            acc[:, t % K] += v
    if case["mean"]:
        if case["vector"]:
            acc /= T
        else:
            acc /= torch.bincount(torch.arange(T) % K, minlength=K).to(dev)
    if case["link"] == "sigmoid":
        acc = torch.sigmoid(acc)
    elif case["link"] == "softmax":
        acc = torch.softmax(acc, 1)
    return {"bins": None, "scores": acc} if case["call"] == "binned" else acc
