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
