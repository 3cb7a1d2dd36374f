"""Ragged trees as padded heaps (packed arrays 14-18): a CPU interpreter of the layout against the
oracle, and the kernel at the edges of its tiles, groups, batches and layouts."""
import numpy as np
import pytest

import oracle
import paper_2405_12491_amd as B
from oracle import binning
from parity_util import assert_scores
from synth import (AGG_MEAN, AGG_SUM, XFORM_IDENTITY, XFORM_SIGMOID, XFORM_SOFTMAX, concat_trees,
                   perfect_tree_arrays, permute_nodes, random_tiny_forest, with_vector_leaves)

GRID = [-1.0, -0.0, 0.0, 0.5, 1.0]
VALUES = np.array([-1.0, -0.0, 0.0, 0.5, 1.0, 2.0, np.nan, np.inf, -np.inf], np.float32)


def batch(levels):
    return 2 if levels == 7 else 4


def walk_heaps(f, X, bins=None):
    """Leaf ids and leaf words of every (row, tree) by the kernel's walk of the layout."""
    binned = bins is not None
    top = B.bridger_forest_packed(f.handle, 17 if binned else 14, np.uint32).reshape(-1, 2)
    blk = B.bridger_forest_packed(f.handle, 18 if binned else 15, np.uint32)
    ids = B.bridger_forest_packed(f.handle, 16, np.int32)
    order = B.bridger_forest_packed(f.handle, 3, np.int32)
    T, n = f.n_trees, X.shape[0]
    L = [l for l in (5, 6, 7) if top.shape[0] == (T + batch(l)) << l]
    assert len(L) == 1
    L = L[0]
    top = top.reshape(-1, 1 << L, 2)
    assert not top[T:].any()
    flat = f.info()["max_depth"] <= L
    s = 7 if binned or f.n_features > 256 else 8
    V = bins if binned else X
    rows = np.arange(n)

    def right(w, x):
        return (x > w.astype(np.int64)) if binned else ~(x <= w.view(np.float32))

    leaves, words = np.empty((n, T), np.int32), np.empty((n, T), np.uint32)
    for k in range(T):
        first = int(top[k, 0, 0])
        m = np.ones(n, np.int64)
        for _ in range(L):
            rec = top[k][m]
            m = 2 * m + right(rec[:, 0].copy(), V[rows, rec[:, 1] >> s])
        if flat:
            i = first + m - (1 << L)
            leaves[:, order[k]], words[:, order[k]] = ids[i], blk[i]
            continue
        b4 = blk.reshape(-1, 4)
        level0, width = first, 1 << L
        done = np.zeros(n, bool)
        for _ in range(30):
            i = np.where(done, first, level0 + m - width)
            q = b4[i]
            b1 = right(q[:, 0].copy(), V[rows, (q[:, 3] >> s) & 1023]).astype(np.int64)
            rot = np.where(b1 == 1, 21, 10).astype(np.uint32)
            m2 = (q[:, 3] >> rot) | (q[:, 3] << (32 - rot))
            wc = np.where(b1 == 1, q[:, 2], q[:, 1]).astype(np.uint32)
            fin = ~done & ((m2 >> s) & 1024 != 0)
            leaves[fin, order[k]] = ids[2 * i[fin] + b1[fin]]
            words[fin, order[k]] = wc[fin]
            done |= fin
            if done.all():
                break
            m = 4 * m + 2 * b1 + right(wc, V[rows, (m2 >> s) & 1023])
            level0, width = level0 + width, 4 * width
        assert done.all()
    return leaves, words


@pytest.mark.parametrize("depth", [0, 1, 4, 5, 6, 7, 8, 9, 10, 11])
def test_heap_layout(depth):
    """Forests of every layout (leaf words below 5, 6 or 7 levels; blocks below 5 or 6), with
    leaves at every level, ties and non-finite inputs: the oracle's leaf ids and values."""
    rng = np.random.default_rng(500 + depth)
    F = int(rng.integers(1, 12))
    model = permute_nodes(random_tiny_forest(rng, 17, F, max_depth=depth, p_split=0.85, thr_grid=GRID), rng)
    X = rng.choice(VALUES, (96, F))
    _, ref_lv, _ = oracle.predict(model, X, want_leaves=True)
    ref_val = model.value[model.tree_offsets[:-1][None, :] + ref_lv].astype(np.float32)
    with B.Forest(model, host_only=True) as f:
        f.kernel = B.BRIDGER_KERNEL_RAGGED
        for bins in (None, binning.bin_rows(binning.tables(model), X)):
            lv, words = walk_heaps(f, X, bins)
            assert np.array_equal(lv, ref_lv)
            assert np.array_equal(words.view(np.float32), ref_val)


@pytest.mark.parametrize("kind", ["normal", "tail", "few", "wide", "denormal", "infinite"])
@pytest.mark.parametrize("perfect", [False, True])
def test_ranks_of_any_thresholds(kind, perfect):
    """The tables of thresholds (packed arrays 5 and 6; long ones are sorted by their bits) are the sorted
    distinct ones, and the heaps of ranks lead bins to the oracle's leaves, whatever the spread."""
    rng = np.random.default_rng(len(kind))
    draw = {"normal": rng.standard_normal, "tail": lambda n: np.exp(9 * rng.standard_normal(n)) * rng.choice([-1, 1], n),
            "few": lambda n: rng.choice([-1.5, -0.0, 0.0, 2.0], n), "wide": lambda n: rng.uniform(-3.4e38, 3.4e38, n),
            "denormal": lambda n: rng.integers(-9, 9, n) * 1e-45,
            "infinite": lambda n: np.where(rng.random(n) < 0.1, rng.choice([-np.inf, np.inf], n), rng.standard_normal(n))}[kind]
    F = 2
    if perfect:
        trees = [perfect_tree_arrays(7, rng.integers(0, F, 127), draw(127).astype(np.float32),
                                     rng.standard_normal(128).astype(np.float32)) for _ in range(40)]
        model = concat_trees(trees, F)
    else:
        model = random_tiny_forest(rng, 40, F, max_depth=8, p_split=0.9)
        model.threshold[:] = np.where(model.left >= 0, draw(model.n_nodes), 0.0).astype(np.float32)
    tables = binning.tables(model)
    X = np.concatenate([rng.choice(np.concatenate([t, np.nextafter(t, np.float32(np.inf)), VALUES]), (200, 1))
                        for t in tables], 1).astype(np.float32)
    _, ref_lv, _ = oracle.predict(model, X, want_leaves=True)
    with B.Forest(model, host_only=True) as f:
        values = B.bridger_forest_packed(f.handle, 5, np.float32)
        off = B.bridger_forest_packed(f.handle, 6, np.int32)
        f.kernel = B.BRIDGER_KERNEL_RAGGED
        lv, _ = walk_heaps(f, X, binning.bin_rows(tables, X))
    for i, t in enumerate(tables):
        assert np.array_equal(values[off[i]:off[i + 1]], t)
    assert kind in ("few", "denormal") or np.diff(off).min() > 1024
    assert np.array_equal(lv, ref_lv)


def test_heap_layout_vector_leaves():
    """Vector leaves: a leaf's word is its place among the leaf records."""
    rng = np.random.default_rng(7)
    model = with_vector_leaves(random_tiny_forest(rng, 9, 5, max_depth=10, p_split=0.85), 3, rng)
    X = rng.standard_normal((64, 5)).astype(np.float32)
    with B.Forest(model, host_only=True) as f:
        f.kernel = B.BRIDGER_KERNEL_RAGGED
        lv, words = walk_heaps(f, X)
        rec = B.bridger_forest_packed(f.handle, 0, np.uint32).reshape(-1, 2)
        node = B.bridger_forest_packed(f.handle, 2, np.int32)
        start = B.bridger_forest_packed(f.handle, 1, np.int32)
        leaf_rec = np.flatnonzero(((rec[:, 1] & 0x8000) != 0) & (node >= 0))
        got = leaf_rec[words]
        tree = np.searchsorted(start, got, side="right") - 1
        assert np.array_equal(tree, np.broadcast_to(np.arange(9), tree.shape))
        assert np.array_equal(node[got], lv)


@pytest.mark.parametrize("n_rows,features,rows", [(1, 28, 16), (3001, 28, 16), (4096, 28, 16), (4097, 28, 32),
                                                  (8192, 28, 32), (8193, 28, 64), (10**6, 28, 64), (10**6, 256, 64),
                                                  (3000, 600, 16), (5000, 600, 32), (10**6, 600, 32)])
def test_heap_plan_fits(n_rows, features, rows):
    """Every batch size gets a plan within a CU's LDS: a tile of 64 columns (32 above 256 features) and a
    heap copy per lane group.  The rows of a workgroup reported are those it takes, 16 or 32 in a small
    batch however many columns the tile has, and the bytes count its workgroups."""
    rng = np.random.default_rng(3)
    model = random_tiny_forest(rng, 40, features, max_depth=9)
    with B.Forest(model, host_only=True) as f:
        f.kernel = B.BRIDGER_KERNEL_RAGGED
        p = f.plan(n_rows)
        columns = 64 if features <= 256 else 32
        assert p["rows_per_wg"] == rows and 0 < p["lds_bytes"] <= 163840
        groups = (p["lds_bytes"] - features * columns * 4) // 2048  # 6 top levels: 2 KB a group
        assert groups in (1, 2, 4, 8, 16, 32, 64)
        staged = B.bridger_forest_packed(f.handle, 0, np.uint8).size / 4.0  # per workgroup
        big = 1 << 20
        walk = (f.plan(big)["lds_read_bytes"] - big // columns * staged) / big  # per row
        assert p["lds_read_bytes"] == pytest.approx(n_rows * walk + -(-n_rows // rows) * staged)


@pytest.mark.gpu
@pytest.mark.parametrize("F", [256, 257, 577, 1023])
@pytest.mark.parametrize("waves,rows", [(0, 0), (1, 32), (8, 32), (4, 16), (8, 16)])
def test_wide_rows(F, waves, rows, monkeypatch):
    """Tiles of 64 and of 32 columns (above 256 features): dense rows, CSR rows, a scaler, leaf ids,
    several classes and vector leaves."""
    import dataclasses

    import torch

    from oracle import vector
    if waves:
        monkeypatch.setenv("BRIDGER_WAVES", str(waves))
        monkeypatch.setenv("BRIDGER_HEAP_ROWS", str(rows))
    rng = np.random.default_rng(F)
    base = random_tiny_forest(rng, 70, F, max_depth=8, p_split=0.9)
    models = [base, dataclasses.replace(base, n_classes=5, transform=XFORM_SOFTMAX), with_vector_leaves(base, 3, rng)]
    n = 70
    X = rng.standard_normal((n, F)).astype(np.float32)
    X[rng.random((n, F)) < 0.5] = 0.0
    mean, scale = rng.normal(0, 0.2, F), rng.uniform(0.8, 1.2, F)
    Xs = ((X.astype(np.float64) - mean).astype(np.float32).astype(np.float64) / scale).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    nz = (Xd != 0)
    csr = (torch.cat([torch.zeros(1, dtype=torch.int64, device="cuda"), nz.sum(1).cumsum(0)]),
           nz.nonzero()[:, 1].to(torch.int32), Xd[nz])
    for model in models:
        predict = vector.predict if model.value.ndim == 2 else \
            (lambda m, x: oracle.predict(m, x, want_leaves=True)[:2])
        ref, ref_lv = predict(model, X)
        refs, _ = predict(model, Xs)
        with B.Forest(model) as f:
            print(f"F={F} {waves}x{rows} K={model.n_classes} plan {f.plan(n)}", flush=True)
            assert_scores(f.predict(Xd).cpu().numpy(), ref, "dense")
            assert_scores(f.predict_csr(*csr, n).cpu().numpy(), ref, "csr")
            assert np.array_equal(f.predict_leaves(Xd).cpu().numpy(), ref_lv)
            f.set_preprocess(B.BRIDGER_PRE_CENTER_SCALE, mean, scale)
            assert_scores(f.predict(Xd).cpu().numpy(), refs, "scaled")


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [0, 16, 32])
@pytest.mark.parametrize("F", [1, 7, 28, 256, 300, 784])
def test_normalizer_from_the_tile(F, rows, monkeypatch):
    """The Normalizer inside the walk: every threshold is some row's normalized value, so a last-bit
    error anywhere changes a leaf; a zero row, a NaN row and an infinite one among them."""
    import torch

    from oracle import preprocess as P
    if rows:
        monkeypatch.setenv("BRIDGER_HEAP_ROWS", str(rows))
    rng = np.random.default_rng(F)
    n = 150
    X = (rng.standard_normal((n, F)) * np.exp(rng.standard_normal((n, 1)))).astype(np.float32)
    X[3], X[5, 0], X[7, F - 1] = 0.0, np.nan, np.inf
    with np.errstate(invalid="ignore"):
        Xn = P.apply(P.NORMALIZE, None, None, X)
    model = random_tiny_forest(rng, 40, F, max_depth=9, p_split=0.9)
    pool = Xn[rng.integers(8, n, model.n_nodes), np.maximum(model.feature, 0)]
    model.threshold[:] = np.where(model.left >= 0, pool, 0.0)
    ref, ref_lv, _ = oracle.predict(model, Xn, want_leaves=True)
    Xd = torch.from_numpy(X).cuda()
    with B.Forest(model) as f:
        f.kernel = B.BRIDGER_KERNEL_RAGGED
        f.set_preprocess(B.BRIDGER_PRE_NORMALIZE)
        assert np.array_equal(f.predict_leaves(Xd).cpu().numpy(), ref_lv)
        assert_scores(f.predict(Xd).cpu().numpy(), ref, f"normalized F={F}")


@pytest.mark.gpu
@pytest.mark.parametrize("n_rows", [1, 17, 4096, 4097, 8193, 131072, 131073])
def test_perfect_small_batches(n_rows):
    """AUTO on perfect forests around the rows where the shape of the walk changes (16-, 32- and
    64-row groups, then the PERFECT kernels): the explicit PERFECT kernel's outputs."""
    import torch
    rng = np.random.default_rng(n_rows)
    # (trees of few levels or leaves stay with PERFECT, whatever the batch)
    for D, K, T, walk in ((3, 1, 129, False), (3, 1, 128, False), (6, 1, 20, False), (6, 3, 70, True), (8, 1, 40, True)):
        trees = [perfect_tree_arrays(D, rng.integers(0, 10, (1 << D) - 1),
                                     rng.standard_normal((1 << D) - 1).astype(np.float32),
                                     rng.standard_normal(1 << D).astype(np.float32)) for _ in range(T)]
        model = concat_trees(trees, 10, K, None if K == 1 else np.arange(T) % K, AGG_SUM,
                             XFORM_SIGMOID if K == 1 else XFORM_SOFTMAX)
        X = torch.from_numpy(rng.standard_normal((n_rows, 10)).astype(np.float32)).cuda()
        with B.Forest(model) as f:
            assert f.kernel == B.BRIDGER_KERNEL_PERFECT
            q = f.bin(X)
            got = [f.predict(X), f.predict_binned(q), f.predict_labels(X), f.predict_leaves(X)]
            assert (f.plan(n_rows)["chunk_bytes"] == 0) == (n_rows <= 131072 and walk)
            f.kernel = B.BRIDGER_KERNEL_PERFECT
            ref = [f.predict(X), f.predict_binned(q), f.predict_labels(X), f.predict_leaves(X)]
            assert f.plan(n_rows)["chunk_bytes"] > 0
        for g, r in zip(got[:2], ref[:2]):  # double sums in another order, rounded once
            assert torch.allclose(g, r, rtol=2.4e-7, atol=1e-7)
        assert torch.equal(got[2], ref[2]) and torch.equal(got[3], ref[3])


@pytest.mark.parametrize("D,T,F,n,walk", [
    (4, 1000, 28, 40_000, False), (1, 897, 71, 167_000, False), (3, 1125, 21, 671, True), (4, 164, 157, 116_000, True),
    (6, 100, 28, 10_000, True), (8, 18, 16, 33_000, True), (7, 18, 16, 33_000, False), (8, 8, 58, 90_000, False),
    (8, 5, 226, 252_000, False), (8, 5, 228, 252_000, True), (6, 43, 250, 240_000, False), (6, 463, 209, 200_000, True),
    (5, 281, 195, 2_309, False), (6, 95, 18, 59_458, False),
    (6, 95, 18, 29_000, True), (5, 143, 300, 77_537, False), (5, 143, 299, 77_537, True), (6, 500, 28, 1_000, True), (6, 500, 28, 1_000_000, False)])
def test_perfect_walk_rule(D, T, F, n, walk):
    """Which perfect forests AUTO gives to the padded-heap walk (no chunks in the plan): on both sides of
    each clause, the shapes on which it was measured."""
    rng = np.random.default_rng(D)
    trees = [perfect_tree_arrays(D, rng.integers(0, F, (1 << D) - 1), rng.standard_normal((1 << D) - 1).astype(np.float32),
                                 np.zeros(1 << D, np.float32)) for _ in range(T)]
    with B.Forest(concat_trees(trees, F), host_only=True) as f:
        assert f.kernel == B.BRIDGER_KERNEL_PERFECT
        assert (f.plan(n)["chunk_bytes"] == 0) == walk


@pytest.mark.gpu
@pytest.mark.parametrize("F", [28, 63, 64, 300])
@pytest.mark.parametrize("T", [1, 3, 16, 17])
def test_few_trees(T, F):
    """Ragged forests with fewer trees than waves that load the row tile, around the batch sizes where
    the lane groups change, against the oracle."""
    import torch
    rng = np.random.default_rng(100 * T + F)
    model = random_tiny_forest(rng, T, F, max_depth=9, p_split=0.9)
    X = rng.standard_normal((8193, F)).astype(np.float32)
    ref, ref_lv, _ = oracle.predict(model, X, want_leaves=True)
    Xd = torch.from_numpy(X).cuda()
    with B.Forest(model) as f:
        f.kernel = B.BRIDGER_KERNEL_RAGGED
        for n in (1, 4097, 8193):
            what = f"F={F} T={T} rows={n} plan {f.plan(n)}"
            print(what, flush=True)
            assert_scores(f.predict(Xd[:n]).cpu().numpy(), ref[:n], what)
            assert np.array_equal(f.predict_leaves(Xd[:n]).cpu().numpy(), ref_lv[:n]), what


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [64, 32, 16])
@pytest.mark.parametrize("waves", [1, 2, 8, 16])
@pytest.mark.parametrize("depth", [3, 6, 7, 8, 9, 12])
def test_heap_kernel(depth, waves, rows, monkeypatch):
    """Scores, labels, leaf ids, bins and CSR rows around the tile's edges, for every number of
    lane groups, scalar leaves of 1, 3 and 13 classes and vector leaves of 2, 7 and 9."""
    import dataclasses

    import torch

    from oracle import vector
    # (this walk's waves alone: a record plan of one wave has no 128-row tile for 8-bit bins)
    monkeypatch.setenv("BRIDGER_HEAP_WAVES", str(waves))
    monkeypatch.setenv("BRIDGER_HEAP_ROWS", str(rows))
    rng = np.random.default_rng(900 + depth)
    F = 7 if depth % 2 else 12
    T = 17 if depth != 8 else 71
    grid = GRID if depth != 9 else None
    base = random_tiny_forest(rng, T, F, max_depth=depth, p_split=0.9, thr_grid=grid)
    models = [dataclasses.replace(base, transform=XFORM_SIGMOID)]
    for K in (3, 13):
        models.append(dataclasses.replace(base, n_classes=K, aggregate=AGG_MEAN, transform=XFORM_SOFTMAX,
                                          base_score=rng.standard_normal(K).astype(np.float32)))
    models += [with_vector_leaves(base, 2, rng), with_vector_leaves(base, 7, rng),
               with_vector_leaves(base, 9, rng, AGG_SUM, XFORM_IDENTITY)]
    for model in models:
        for n in (1, 63, 65):
            X = rng.choice(VALUES[:7], (n, F)) if grid else rng.standard_normal((n, F)).astype(np.float32)
            what = f"depth {depth} waves {waves}x{rows} K {model.n_classes} rows {n}"
            print(what, flush=True)
            if model.value.ndim == 2:
                ref, ref_lv = vector.predict(model, X)
            else:
                ref, ref_lv, _ = oracle.predict(model, X, want_leaves=True)
            Xd = torch.from_numpy(X).cuda()
            with B.Forest(model) as f:
                f.kernel = B.BRIDGER_KERNEL_RAGGED
                q = f.bin(Xd)
                idx = np.tile(np.arange(F, dtype=np.int32), n)
                csr = (torch.arange(0, n * F + 1, F).cuda(), torch.from_numpy(idx).cuda(), Xd.reshape(-1))
                outs = [f.predict(Xd), f.predict_csr(*csr, n), f.predict_binned(q)]
                lvs = [f.predict_leaves(Xd), f.predict_csr(*csr, n, leaves=True), f.predict_binned_leaves(q)]
                torch.cuda.synchronize()
            for o in outs:
                assert_scores(o.cpu().numpy(), ref, what)
            for l in lvs:
                assert np.array_equal(l.cpu().numpy(), ref_lv), what


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [8, 16])
@pytest.mark.parametrize("depth", [6, 9, 10])
def test_binned_tables(depth, bits):
    """Bins of a whole table of narrow rows, in the plan that the walk takes by itself there (one wave
    of 64 rows a workgroup): scores and leaf ids, 8- and 16-bit bins, one class, several, vector leaves."""
    import dataclasses

    import torch

    from oracle import vector
    rng = np.random.default_rng(10 * depth + bits)
    F, n = 3, (1 << 19) + 77
    base = random_tiny_forest(rng, 12 if bits == 8 else 30, F, max_depth=depth, p_split=0.95,
                              thr_grid=GRID if bits == 8 else None)
    X = rng.choice(VALUES[:7], (n, F)) if bits == 8 else rng.standard_normal((n, F)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    for model in (base, dataclasses.replace(base, n_classes=3, transform=XFORM_SOFTMAX), with_vector_leaves(base, 7, rng)):
        if model.value.ndim == 2:
            ref, ref_lv = vector.predict(model, X, threads=8)
        else:
            ref, ref_lv, _ = oracle.predict(model, X, want_leaves=True, threads=8)
        with B.Forest(model) as f:
            f.kernel = B.BRIDGER_KERNEL_RAGGED
            q = f.bin(Xd)
            what = f"depth {depth} {q.dtype} K {model.n_classes}"
            print(what, flush=True)
            assert q.element_size() * 8 == bits
            assert_scores(f.predict_binned(q).cpu().numpy(), ref, what)
            assert np.array_equal(f.predict_binned_leaves(q).cpu().numpy(), ref_lv), what


@pytest.mark.gpu
@pytest.mark.parametrize("depth,K,T", [(8, 13, 20), (10, 32, 96), (8, 39, 39)])
def test_bins_of_few_trees_a_class(depth, K, T):
    """Bins of many classes of few trees, in batches of each plan."""
    import dataclasses

    import torch
    rng = np.random.default_rng(K)
    F = 4
    model = dataclasses.replace(random_tiny_forest(rng, T, F, max_depth=depth, p_split=0.9), n_classes=K,
                                transform=XFORM_SOFTMAX, base_score=rng.standard_normal(K).astype(np.float32))
    X = rng.standard_normal((40_001, F)).astype(np.float32)
    ref, ref_lv, _ = oracle.predict(model, X, want_leaves=True, threads=8)
    Xd = torch.from_numpy(X).cuda()
    with B.Forest(model) as f:
        assert f.kernel == B.BRIDGER_KERNEL_RAGGED
        for n in (1, 1000, 40_001):
            q = f.bin(Xd[:n])
            print(f"K={K} T={T} rows={n} {q.dtype}", flush=True)
            assert_scores(f.predict_binned(q).cpu().numpy(), ref[:n], f"K={K} rows={n}")
            assert np.array_equal(f.predict_binned_leaves(q).cpu().numpy(), ref_lv[:n])


@pytest.mark.gpu
@pytest.mark.parametrize("K,F,agg", [(2, 5, AGG_MEAN), (8, 5, AGG_SUM), (9, 5, AGG_MEAN), (33, 90, AGG_SUM), (60, 160, AGG_MEAN),
                                     (64, 5, AGG_SUM)])
def test_softmax_of_many_classes(K, F, agg):
    """The classes of a row shared by its lane groups: fewer classes than groups, as many, more; groups of 16 and 32
    rows, 2 waves of the former where the sums of 4 do not fit, and 64-row groups of few waves."""
    import dataclasses

    import torch
    rng = np.random.default_rng(K)
    base = rng.standard_normal(K).astype(np.float32)
    base[0] = -np.inf  # the first class's score, from which the maximum starts
    model = dataclasses.replace(random_tiny_forest(rng, 2 * K + 1, F, max_depth=8, p_split=0.9), n_classes=K, aggregate=agg,
                                transform=XFORM_SOFTMAX, base_score=base)
    X = rng.standard_normal((30_001, F)).astype(np.float32)
    ref, _, _ = oracle.predict(model, X, threads=8)
    assert np.isfinite(ref).all() and not ref[:, 0].any()
    Xd = torch.from_numpy(X).cuda()
    with B.Forest(model) as f:
        assert f.kernel == B.BRIDGER_KERNEL_RAGGED
        for n in (1, 130, 4096, 5003, 30_001):
            print(f"K={K} rows={n}", flush=True)
            assert_scores(f.predict(Xd[:n]).cpu().numpy(), ref[:n], f"K={K} rows={n}")
            assert_scores(f.predict_binned(f.bin(Xd[:n])).cpu().numpy(), ref[:n], f"bins K={K} rows={n}")
