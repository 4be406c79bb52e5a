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


def _three_kinds(n, d, tight, seed):
    """Rows of eight wide groups (half precision certifies them: the k-th and the k'-th neighbour are some ten times as far
    apart as its bound), a share `tight` of rows of eight groups a fifth as wide (it does not, three products do), and two
    rows with 200 copies each, more than k' (the exact pass).  tight: the shares of the two halves."""
    rng = np.random.default_rng(seed)
    narrow = rng.random(n) < np.where(np.arange(n) < n // 2, *tight)
    X = rng.standard_normal((16, d))[rng.integers(0, 8, n) + 8 * narrow]
    X += np.where(narrow, 0.2, 1.0)[:, None] * rng.standard_normal((n, d))
    copies = rng.choice(np.flatnonzero(~narrow), 400, replace=False)
    X[copies] = X[copies[np.arange(400) % 2]]
    rows = np.concatenate([copies[:10], np.flatnonzero(narrow)[::500], np.arange(0, n, n // 40)])
    return X.astype(np.float32), np.unique(rows)


@pytest.mark.parametrize("n,d,tight,half_launches,passes", [
    (33000, 72, (0.3, 0.3), 17, 2),      # one block of query rows, and the second sweep
    (33000, 200, (0.3, 0.3), 17, 2),
    (33000, 300, (0.3, 0.3), 17, 2),     # (buffers of its own)
    (66000, 80, (0.3, 0.3), 66, 3),      # two blocks
    (66000, 80, (0.6, 0.0), 33, 3),      # a first block that is mostly narrow: the next one does without
])
def test_half_precision_sweep(n, d, tight, half_launches, passes):
    """Query tile by query tile, from 32,768 rows on; what it cannot certify goes on to three products and the exact pass."""
    from helpers import launches
    k = 90
    if d < 256:     # the buffers have to fit where rows of P are sorted later, or the sweep is not taken
        block = min(n, 65536)
        assert 2 * n * ((d + 63) // 64 * 64) + 4 * block * ((d + 31) // 32 * 32) + 4 * block + 768 <= 16 * n * k
    X, rows = _three_kinds(n, d, tight, seed=n + d)
    _, count = launches(lambda: _check_against_oracle(X, 30.0, k, rows=rows))
    assert count["knn_tile_half"] == half_launches
    blocks = half_launches // ((n + 2047) // 2048)
    assert count["knn_tile_half<true,false>"] == blocks         # the first launch of a block keeps every pair
    assert count["knn_tile_half<false,true>"] == half_launches - blocks
    assert count["knn_rerank"] == passes
    assert count["knn_exact_select"] >= 400 // (2 * k)


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
