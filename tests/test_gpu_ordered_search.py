"""The exact search in an order of the rows (from 196,608 rows of up to 64 coordinates in groups well apart), against the oracle:
lists bit for bit on sampled rows, P to its float, and which way the rows went."""
import numpy as np
import pytest

from helpers import launches
from test_gpu_build_p import _check_against_oracle

pytestmark = pytest.mark.gpu


def _groups(n, d, groups, scale, seed):
    rng = np.random.default_rng(seed)
    label = rng.integers(0, groups, n)
    X = scale * rng.standard_normal((groups, d))[label] + rng.standard_normal((n, d))
    return X.astype(np.float32), label


@pytest.mark.parametrize("case", ["blobs", "ragged", "one_slab_sorted_ties", "too_few_rows", "touching", "many_tile_borders",
                                  "one_row_far_out", "no_room"])
def test_search(case):
    n, d, groups, scale, k = 196_608, 50, 4, 10.0, 30
    if case == "ragged":
        n, d, groups = 262_145, 64, 3
    if case in ("one_slab_sorted_ties", "no_room"):
        n, d = 200_001, 30
    if case == "too_few_rows":
        n -= 1
    if case == "touching":
        groups, scale = 50, 1.0
    if case == "many_tile_borders":
        d, groups = 8, 20
    if case == "no_room":
        k = 1
    X, label = _groups(n, d, groups, scale, seed=n + d)
    if case == "one_slab_sorted_ties":
        X = X[np.argsort(label, kind="stable")]
        X[1000:1400] = X[1000]                                  # more copies than k': the exact pass
        X[150_000:170_000:40] = X[150_000:170_000:40][:250].repeat(2, axis=0)
    if case == "one_row_far_out":
        X[77_777] = 1e18
    rows = np.unique(np.concatenate([np.arange(0, n, n // 25), [0, 1000, 1399, 77_777, n - 1]]))
    _, count = launches(lambda: _check_against_oracle(np.ascontiguousarray(X), max(1.0, k / 3.0), k, rows=rows))
    ns = 1 if d <= 32 else 2
    along = count[f"knn_tile_resident<{ns},false,true>"]
    if case in ("blobs", "ragged", "one_slab_sorted_ties"):
        assert along > 0 and count[f"knn_tile_resident<{ns},false,false>"] == 0
        assert along < count[f"knn_tile_resident<{ns},true,true>"] * (n // 2048)
    elif case == "many_tile_borders":                            # tried on the first block of query rows, and left
        assert count[f"knn_tile_resident<{ns},true,true>"] == 1 and count[f"knn_tile_resident<{ns},false,false>"] > 0
    elif case != "one_row_far_out":
        assert along == 0 and count[f"knn_tile_resident<{ns},false,false>"] > 0


@pytest.mark.parametrize("case", ["blobs", "ragged", "uneven", "one_slab_sorted_ties", "later_blocks_touch"])
def test_every_list(case):
    """All n lists, those of the query tiles that straddle two groups among them (they are swept by themselves), against the
    same rows with columns of zeros up to 72, which go another way: no order, half precision first.  Distances are the same to
    the bit.  later_blocks_touch: a compact group far away comes first in the order, groups that touch after it."""
    import torch
    from paper_1807_11824_amd import build_P
    n, d, k = 196_608, 50, 30
    if case == "ragged":
        n, d = 262_145, 64
    if case in ("one_slab_sorted_ties", "later_blocks_touch"):
        d = 30 if case == "one_slab_sorted_ties" else 16
    X, label = _groups(n, d, 3 if case == "ragged" else 4, 10.0, seed=7 * n + d)
    if case == "uneven":                    # one group of half the rows, one of 300
        X, label = _groups(n, d, 16, 10.0, seed=5)
        X[: n // 2] -= X[: n // 2].mean(axis=0) - 30.0
        X[:n // 2] = np.random.default_rng(1).standard_normal((n // 2, d)) + 30.0
        X[n // 2: n // 2 + 300] = np.random.default_rng(2).standard_normal((300, d)) - 40.0
    if case == "one_slab_sorted_ties":
        X = X[np.argsort(label, kind="stable")]
        X[1000:1400] = X[1000]
    if case == "later_blocks_touch":
        X, _ = _groups(n, d, 60, 10.0, seed=3)
        X[:66_000] = np.random.default_rng(4).standard_normal((66_000, d)) + 12.0
        order = np.random.default_rng(6).permutation(n - 1) + 1
        X[1:] = X[order]                    # (row 0, the first pivot, is in the compact group)
    X = torch.from_numpy(np.ascontiguousarray(X, np.float32)).to("cuda:0")
    wide = torch.zeros((n, 72), device="cuda:0")
    wide[:, :d] = X
    got, count = launches(lambda: build_P(X, 10.0, k, want_knn=True))
    want = build_P(wide, 10.0, k, want_knn=True)
    assert torch.equal(got["knn_idx"], want["knn_idx"]) and torch.equal(got["knn_d2"], want["knn_d2"])
    ns = 1 if d <= 32 else 2
    alone = count["knn_tile_mfma<4,false,false,false>"]
    if case == "later_blocks_touch":
        assert count[f"knn_tile_resident<{ns},true,true>"] > 1 and count[f"knn_tile_resident<{ns},false,false>"] > 0
        assert count[f"knn_tile_resident<{ns},true,false>"] == 0
    elif case != "uneven":                 # (the half of all rows in one group cannot leave enough out)
        assert count[f"knn_tile_resident<{ns},false,true>"] > 0 and count[f"knn_tile_resident<{ns},false,false>"] == 0
    if case in ("blobs", "ragged"):
        assert alone > 0
