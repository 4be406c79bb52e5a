"""The passes of tsne_build_P at the sizes where they change form, against the oracle (lists bit for bit, P to its float).

Candidates kept per row (k' = k + max(32, k/2): a lane of the compaction holds 8 pairs up to 320, 16 up to 832, 64 beyond);
the first launch of 2048 database rows, which keeps every pair; rows whose sixteen lanes have nothing or something left
over; distances that do not fit the LDS (k > 480); rows of P longer than the 4096 entries sorted in LDS at a time.
"""
import numpy as np
import pytest

from test_gpu_build_p import _check_against_oracle

pytestmark = pytest.mark.gpu


def _blobs(n, d, seed, groups=5):
    rng = np.random.default_rng(seed)
    means = 4.0 * rng.standard_normal((groups, d))
    return (means[rng.integers(0, groups, n)] + rng.standard_normal((n, d))).astype(np.float32)


@pytest.mark.parametrize("k", [1, 5, 90, 300, 500, 700, 1200])
def test_candidates_kept(k):
    _check_against_oracle(_blobs(3000, 20, seed=k), max(1.0, k / 3.0) if k > 1 else 1.0, k)


@pytest.mark.parametrize("n", [100, 2047, 2048, 2049, 2177])
@pytest.mark.parametrize("d", [7, 50, 100, 257, 300])
def test_first_launch(n, d):
    _check_against_oracle(_blobs(n, d, seed=n + d), 10.0, 30)


@pytest.mark.parametrize("d", [30, 50])
def test_first_launch_resident(d):
    _check_against_oracle(_blobs(16500, d, seed=d), 10.0, 30, rows=np.arange(0, 16500, 300))


@pytest.mark.parametrize("d", [20, 100, 300])
def test_ties_at_the_cut(d):
    """A hundred copies of every point: the k'-th distance is shared by many pairs."""
    X = np.repeat(_blobs(30, d, seed=d), 100, axis=0)
    X[::7] += 1.0
    _check_against_oracle(np.ascontiguousarray(X), 10.0, 30)


@pytest.mark.parametrize("d", [20, 300])
def test_distances_beyond_single_precision(d):
    X = _blobs(2500, d, seed=d)
    X[5] = 1e18
    X[2400] = -1e18
    _check_against_oracle(X, 10.0, 30)


@pytest.mark.parametrize("n", [4000, 4097, 4200, 9001])
def test_hub_rows(n):
    """Points on a sphere and two near its centre: everybody lists those two."""
    rng = np.random.default_rng(n)
    X = rng.standard_normal((n, 50))
    X /= np.linalg.norm(X, axis=1, keepdims=True)
    X[[n // 3, n // 2]] *= 0.01
    g = _check_against_oracle(X.astype(np.float32), 4.0, 10)
    assert np.diff(g["row_ptr"])[[n // 3, n // 2]].min() >= n - 50


@pytest.mark.parametrize("n,d,spread", [(33000, 72, 4.0), (33000, 200, 4.0), (33000, 72, 400.0), (66000, 80, 400.0)])
def test_half_precision_sweep_of_shorter_rows(n, d, spread):
    """From 32,768 rows on; far groups leave it without certificates (second sweep), copies those without any (exact pass)."""
    rng = np.random.default_rng(n + d)
    X = spread * rng.standard_normal((8, d))[rng.integers(0, 8, n)] + rng.standard_normal((n, d))
    X[100:500] = X[rng.integers(1000, 1004, 400)]
    rows = np.concatenate([np.arange(100, 500, 50), np.arange(0, n, n // 40)])
    _check_against_oracle(X.astype(np.float32), 10.0, 40, rows=np.unique(rows))


def test_rows_that_three_products_cannot_certify_are_not_swept_twice():
    """Two blocks of query rows.  Half precision certifies none of the first block's (groups far apart against the steps
    between neighbours), so the second block goes through three products, which cannot certify its rows either (a hundred
    copies of each): those are for the exact pass.  The second sweep is for the first block's rows only: one pass, not two."""
    from helpers import launches
    rng = np.random.default_rng(5)
    n, d, k, split = 66000, 256, 20, 33024
    X = 8.0 * rng.standard_normal((8, d))[rng.integers(0, 8, n)] + rng.standard_normal((n, d))
    X[split:] = X[split:][rng.permutation(np.arange(n - split) % 329)]
    X = X.astype(np.float32)
    rows = np.concatenate([np.arange(0, split, split // 30), np.arange(split, n, (n - split) // 10)])
    _, count = launches(lambda: _check_against_oracle(X, 5.0, k, rows=rows))
    assert count["knn_tile_half"] == (n + 2047) // 2048         # the first block's launches
    assert count["knn_exact_select"] > 100                      # (2 k rows a launch)
    assert count["knn_rerank"] == 3                             # two blocks, one pass of the second sweep


def test_half_precision_is_not_tried_on_points_near_a_plane():
    """Neighbours closer together than half precision can tell: the sweep would certify no row, and the lists need the
    three-product tiles anyway."""
    from helpers import launches
    rng = np.random.default_rng(7)
    n, d = 33000, 72
    X = (rng.random((n, 2)) @ rng.standard_normal((2, d))).astype(np.float32)
    _, count = launches(lambda: _check_against_oracle(X, 30.0, 90, rows=np.arange(0, n, n // 40)))
    assert count["knn_tile_half"] == 0 and count["knn_tile_mfma"] == (n + 2047) // 2048
