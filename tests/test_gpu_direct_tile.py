"""The DIRECT tile kernel (pair records, features from an LDS tile) against the oracle: every number
of waves its plan can take, batches with a remainder, and forests that only DIRECT can take."""
import dataclasses

import numpy as np
import pytest

import oracle
import paper_2405_12491_amd as B
from oracle import vector
from parity_util import assert_scores
from synth import (AGG_MEAN, XFORM_SIGMOID, XFORM_SOFTMAX, permute_nodes, random_tiny_forest,
                   with_vector_leaves)

pytestmark = pytest.mark.gpu
GRID = [-1.0, -0.0, 0.0, 0.5, 1.0]
VALUES = np.array([-1.0, -0.0, 0.0, 0.5, 1.0, 2.0, np.nan, np.inf, -np.inf], np.float32)


def check(model, X, what, exact, rows=64):
    import torch
    print(what, flush=True)
    if model.value.ndim == 2:
        ref, ref_lv = vector.predict(model, X)
    else:
        ref, ref_lv, _ = oracle.predict(model, X, want_leaves=True)
    Xd = torch.from_numpy(X).cuda()
    with B.Forest(model) as f:
        f.kernel = B.BRIDGER_KERNEL_DIRECT
        assert f.plan(X.shape[0])["rows_per_wg"] == rows
        out = f.predict(Xd).cpu().numpy()
        lv = f.predict_leaves(Xd).cpu().numpy()
    assert np.array_equal(lv, ref_lv), what
    assert_scores(out, ref, what)
    if exact:  # trees are added one after the other, in the caller's order per class
        assert np.array_equal(out, ref.astype(np.float32)), what


@pytest.mark.parametrize("tile", ["1", "2"])
@pytest.mark.parametrize("trees", [1, 3, 4, 5, 9, 33, 64, 65, 131])
def test_direct_tile(trees, tile, monkeypatch):
    """The tile (1), and the same records row by row (2)."""
    monkeypatch.setenv("BRIDGER_DIRECT_TILE", tile)
    rng = np.random.default_rng(40 + trees)
    F = 5 if trees % 2 else 8
    base = permute_nodes(random_tiny_forest(rng, trees, F, max_depth=9, p_split=0.85, thr_grid=GRID), rng)
    models = [(base, True), (dataclasses.replace(base, transform=XFORM_SIGMOID, aggregate=AGG_MEAN), False)]
    for K in (2, 11):
        models.append((dataclasses.replace(base, n_classes=K, transform=XFORM_SOFTMAX,
                                           base_score=rng.standard_normal(K).astype(np.float32)), False))
    for K in (2, 6, 64):
        models.append((with_vector_leaves(base, K, rng), False))
    for model, exact in models:
        for n in (1, 64, 129):
            check(model, rng.choice(VALUES, (n, F)), f"{trees} trees K {model.n_classes} rows {n}", exact,
                  64 if tile == "1" else 256)


@pytest.mark.parametrize("trees,F", [(6, 9), (1, 9), (3, 100)])
def test_large_trees(trees, F):
    """Trees of more records than a RAGGED leaf can point over, in the way that the library takes by
    itself (the tile; row by row for few trees), with a fused scaler too."""
    import torch
    rng = np.random.default_rng(4)
    model = random_tiny_forest(rng, trees, F, max_depth=17, p_split=0.97)
    assert np.diff(model.tree_offsets).max() > 40000
    X = rng.standard_normal((700, F)).astype(np.float32)
    with B.Forest(model, host_only=True) as f:
        assert f.kernel == B.BRIDGER_KERNEL_DIRECT
    check(model, X, "large trees", True, 256 if trees == 1 else 64)
    mean, scale = rng.normal(0, 0.2, F), rng.uniform(0.8, 1.2, F)
    Xs = ((X.astype(np.float64) - mean).astype(np.float32).astype(np.float64) / scale).astype(np.float32)
    with B.Forest(model) as f:
        f.set_preprocess(B.BRIDGER_PRE_CENTER_SCALE, mean, scale)
        out = f.predict(torch.from_numpy(X).cuda()).cpu().numpy()
    ref, _, _ = oracle.predict(model, Xs)
    assert_scores(out, ref, "scaled")
