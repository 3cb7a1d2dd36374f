"""The binning kernel's grid cells at their edges: thresholds of any spread (one cell holding most of
them, infinite ones, one or none), staged and in place, with and without 4-column loads."""
import numpy as np
import pytest

import paper_2405_12491_amd as B
from oracle import binning
from synth import concat_trees, perfect_tree_arrays

pytestmark = pytest.mark.gpu


def _forest(rng, tables):
    """Stumps whose thresholds on feature f are tables[f] (a feature may have none)."""
    leaf = np.array([0.0, 1.0], np.float32)
    trees = [perfect_tree_arrays(1, np.array([f]), np.array([t], np.float32), leaf)
             for f, ts in enumerate(tables) for t in ts]
    return concat_trees(trees, len(tables))


def _tables(rng, F, n):
    kinds = [
        lambda: rng.standard_normal(n),
        lambda: np.exp(8 * rng.standard_normal(n)),                       # one cell holds most
        lambda: np.concatenate([rng.random(n) * 1e-30, [1e30, -1e30]]),  # all but two in one cell
        lambda: np.array([-np.inf, -1.0, 0.0, -0.0, 2.0, np.inf]),
        lambda: np.array([-3.0e38, 3.0e38, 0.0]),                         # the range overflows
        lambda: np.array([0.25]),
        lambda: np.array([np.inf]),
        lambda: np.array([]),
        lambda: np.array([1e-45, 2e-45, -1e-45]),                         # denormals
        lambda: np.repeat(rng.integers(0, 5, n), 2).astype(float),
    ]
    return [np.asarray(kinds[(f + F) % len(kinds)](), np.float32) for f in range(F)]


@pytest.mark.parametrize("env", [{"BRIDGER_BIN_KERNEL": "1"}, {"BRIDGER_BIN_KERNEL": "2"},
                                 {"BRIDGER_BIN_KERNEL": "1", "BRIDGER_BIN_LDS_KB": "2"}],
                         ids=lambda e: ",".join(f"{k[8:]}={v}" for k, v in e.items()))
@pytest.mark.parametrize("F,n", [(1, 40), (3, 200), (4, 300), (12, 70), (28, 500), (37, 33), (300, 6), (1100, 2)])
def test_bin_cells(F, n, env, monkeypatch):
    for k, v in env.items():
        monkeypatch.setenv(k, v)
    rng = np.random.default_rng(F * 1000 + n)
    _check(rng, F, _tables(rng, F, n), f"n={n} {env}")


@pytest.mark.parametrize("kernel", ["1", "2"])
@pytest.mark.parametrize("F,n,kb", [(4, 450, 8), (4, 480, 8), (28, 450, 8), (3, 900, 4), (5, 990, 4), (4, 900, 4), (4, 1100, 4)])
def test_coarse_cells(F, n, kb, kernel, monkeypatch):
    """Tables that fit the LDS only with cells of several thresholds (four columns together, one at a
    time, or not at all), staged and in place (there with a cell per threshold)."""
    monkeypatch.setenv("BRIDGER_BIN_LDS_KB", str(kb))
    monkeypatch.setenv("BRIDGER_BIN_KERNEL", kernel)
    rng = np.random.default_rng(n)
    tables = [rng.standard_normal(n) if f % 3 else np.exp(4 * rng.standard_normal(n)) for f in range(F)]
    _check(rng, F, [t.astype(np.float32) for t in tables], f"n={n} {kb} KB kernel {kernel}")


def _check(rng, F, tables, what):
    import torch
    model = _forest(rng, tables)
    rows = 333
    X = rng.standard_normal((rows, F)).astype(np.float32)
    for f, t in enumerate(tables):  # thresholds, their neighbours and the special values
        pool = np.concatenate([t, np.nextafter(t, np.float32(np.inf)), np.nextafter(t, np.float32(-np.inf)),
                               np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, 3.4e38, -3.4e38], np.float32)])
        pick = rng.random(rows) < 0.8
        X[pick, f] = rng.choice(pool, int(pick.sum()))
    ref = binning.bin_rows(binning.tables(model), X)
    with B.Forest(model) as f:
        bb = f.bin_info()["bin_bytes"]
        dt = torch.uint8 if bb == 1 else torch.int16
        for shift in (0, 1):  # rows 16-byte aligned where F allows, and not
            buf = torch.zeros(rows * F + 1, device="cuda")
            Xd = buf[shift:shift + rows * F].view(rows, F)
            Xd.copy_(torch.from_numpy(X))
            qs = shift * 4 // bb  # outputs are 4-byte aligned
            qbuf = torch.zeros(rows * F + 4, dtype=dt, device="cuda")
            q = qbuf[qs:qs + rows * F].view(rows, F)
            print(f"bins F={F} shift={shift} {what}", flush=True)
            B.bridger_forest_bin(f.handle, Xd.data_ptr(), rows, F, q.data_ptr(),
                                 torch.cuda.current_stream().cuda_stream)
            got = q.cpu().numpy().view(np.uint8 if bb == 1 else np.uint16)
            assert np.array_equal(got.astype(np.int64), ref.astype(np.int64))
            assert not qbuf[:qs].any() and not qbuf[qs + rows * F:].any()
