"""Leaf ids of perfect forests as the kernels store them: 16 or 4 trees at a time, remainders of every
kind, the caller's numbering breadth-first or not."""
import numpy as np
import pytest

import oracle
import paper_2405_12491_amd as B
from synth import concat_trees, perfect_tree_arrays, permute_nodes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("features", [5, 28, 60])
@pytest.mark.parametrize("trees", [1, 4, 15, 16, 17, 31, 64, 67])
@pytest.mark.parametrize("depth", [2, 6, 8, 9])
def test_leaf_stores(depth, trees, features, monkeypatch):
    import torch
    monkeypatch.setenv("BRIDGER_SIZED_PLANS", "0")  # the large batches' plan
    rng = np.random.default_rng(depth * 100 + trees)
    ts = [perfect_tree_arrays(depth, rng.integers(0, features, (1 << depth) - 1),
                              rng.standard_normal((1 << depth) - 1).astype(np.float32),
                              rng.standard_normal(1 << depth).astype(np.float32)) for _ in range(trees)]
    n = 1100
    X = rng.standard_normal((n, features)).astype(np.float32)
    Xd = torch.from_numpy(X).cuda()
    for K, permute in ((1, False), (1, True), (3, False)):
        model = concat_trees(ts, features, K, None if K == 1 else np.arange(trees) % K)
        if permute:
            model = permute_nodes(model, rng)
        ref = oracle.predict(model, X, want_leaves=True)[1]
        with B.Forest(model) as f:
            f.kernel = B.BRIDGER_KERNEL_PERFECT
            for rows in (n, 512, 33):
                print(f"leaves depth {depth} trees {trees} F {features} K {K} {permute} rows {rows}", flush=True)
                out = torch.full((rows * trees + 64,), -7, dtype=torch.int32, device="cuda")
                got = f.predict_leaves(Xd[:rows], out[:rows * trees].view(rows, trees)).cpu().numpy()
                assert np.array_equal(got, ref[:rows])
                assert (out[rows * trees:] == -7).all()
            q = f.bin(Xd)
            assert np.array_equal(f.predict_binned_leaves(q).cpu().numpy(), ref)


@pytest.mark.parametrize("depth,trees,K", [(3, 37, 1), (6, 18, 1), (6, 21, 4), (7, 5, 1)])
def test_leaf_stores_large_batch(depth, trees, K):
    """More rows than the batch-size classes hold: four lane groups a tile up to depth 6."""
    import torch
    rng = np.random.default_rng(depth + trees)
    ts = [perfect_tree_arrays(depth, rng.integers(0, 9, (1 << depth) - 1),
                              rng.standard_normal((1 << depth) - 1).astype(np.float32),
                              rng.standard_normal(1 << depth).astype(np.float32)) for _ in range(trees)]
    model = permute_nodes(concat_trees(ts, 9, K, None if K == 1 else np.arange(trees) % K), rng)
    n = (1 << 19) + 77
    X = rng.standard_normal((n, 9)).astype(np.float32)
    ref = oracle.predict(model, X, want_leaves=True, threads=8)[1]
    Xd = torch.from_numpy(X).cuda()
    with B.Forest(model) as f:
        f.kernel = B.BRIDGER_KERNEL_PERFECT
        assert np.array_equal(f.predict_leaves(Xd).cpu().numpy(), ref)
        assert np.array_equal(f.predict_binned_leaves(f.bin(Xd)).cpu().numpy(), ref)
