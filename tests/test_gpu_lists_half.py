"""The inverted-file search and its quantizer with the values in half precision first: the queries that sweep leaves without
a certificate, for a second one with three products or the exact pass, against the oracle (lists bit for bit)."""
import numpy as np
import pytest

from helpers import launches
from oracle import ivf
from test_gpu_ivf import _dev

pytestmark = pytest.mark.gpu


def _three_kinds(n, d, tight, seed):
    """Rows of eight wide groups, a share `tight` (of the two halves) of rows of eight groups a twentieth as wide, whose 20th
    and 52nd neighbours half precision cannot tell apart (squared distances some 0.04 apart, its bound is 2^-10 of squared
    norms of about 2 d), and two rows with 200 copies each, more than k' (the exact pass)."""
    rng = np.random.default_rng(seed)
    narrow = rng.random(n) < np.where(np.arange(n) < n // 2, *tight)
    X = rng.standard_normal((16, d))[rng.integers(0, 8, n) + 8 * narrow]
    X += np.where(narrow, 0.05, 1.0)[:, None] * rng.standard_normal((n, d))
    copies = rng.choice(n, 400, replace=False)
    X[copies] = X[copies[np.arange(400) % 2]]
    rows = np.concatenate([copies[:10], np.flatnonzero(narrow)[::500], np.arange(0, n, n // 40)])
    return X.astype(np.float32), np.unique(rows)


@pytest.mark.parametrize("n,d,tight,three", [
    (9000, 64, (0.3, 0.3), False),       # (up to 64 columns no tiles at all)
    (9000, 65, (0.0, 0.0), False),       # the 400 copies alone: straight to the exact pass
    (9000, 72, (0.3, 0.3), True),        # 2700 queries for the second sweep
    (9001, 200, (1.0, 0.6), True),       # most of them
    (140_000, 72, (0.0, 0.3), True),     # two passes, the second sweep over rows of both
    (140_000, 80, (0.8, 0.8), True),     # a first pass that is mostly narrow: the next one does without
])
def test_search(n, d, tight, three):
    from paper_1807_11824_amd import ivf_knn
    nlist, tau, k = max(24, n // 400), 3, 20
    X, rows = _three_kinds(n, d, tight, seed=n + d)
    rows = rows[:: max(1, len(rows) // 150)]
    C = ivf.kmeans_init(X, nlist)
    want_idx, want_d2 = ivf.ivf_knn(X, C, tau, k, rows=rows)
    (idx, d2), count = launches(lambda: ivf_knn(_dev(X), _dev(C), tau, k))
    assert np.array_equal(idx[rows.tolist()].cpu().numpy(), want_idx)
    assert np.allclose(d2[rows.tolist()].cpu().numpy(), want_d2, rtol=1e-13, atol=1e-300)
    assert (count["knn_tile_half_lists"] > 0) == (d > 64)
    assert (count["knn_tile_mfma"] > 0) == three


@pytest.mark.parametrize("n,nlist", [(20_000, 400), (7000, 400)])
def test_quantizer_of_tight_groups(n, nlist):
    """Fifty centroids in every group, all within half precision's bound: three products for all points (20,000), the exact
    pass (7000).  Means are exact sums here and double sums there, both rounded to float."""
    from paper_1807_11824_amd import ivf_train
    rng = np.random.default_rng(n)
    X = rng.standard_normal((8, 72))[rng.integers(0, 8, n)] + 0.01 * rng.standard_normal((n, 72))
    X = X.astype(np.float32)
    want, _ = ivf.kmeans_train(X, nlist, 2)
    got, count = launches(lambda: ivf_train(_dev(X), nlist, 2).cpu().numpy())
    assert np.abs(got - want).max() <= 1e-6 * np.abs(X).max()
    assert count["knn_tile_half_other"] > 0 and (count["knn_tile_mfma"] > 0) == (n > 8192)


@pytest.mark.parametrize("largest,half", [(1.6e-15, False), (2.0e-15, True), (0.9e15, True), (1.2e15, False)])
def test_magnitudes(largest, half):
    """Values that half precision is for: from 2^-49 = 1.78e-15 on the factor that undoes the scaling is a normal float, and
    below 1e15 squares are finite.  The lists search takes the largest norm for the largest value."""
    import oracle
    from paper_1807_11824_amd import build_P, ivf_knn, ivf_train
    rng = np.random.default_rng(5)
    n, d, k = 3000, 260, 10
    X = rng.standard_normal((12, d))[rng.integers(0, 12, n)] + rng.standard_normal((n, d))
    X -= X.mean(axis=0)
    exact = (X * (largest / np.abs(X).max())).astype(np.float32)
    g, count = launches(lambda: build_P(_dev(exact), 3.0, k, want_knn=True))
    assert (count["knn_tile_half"] > 0) == half
    assert np.array_equal(g["knn_idx"].cpu().numpy(), oracle.knn(exact, k, rows=np.arange(n))[0])
    lists = (X * (largest / np.sqrt((X * X).sum(axis=1).max()))).astype(np.float32)
    C = ivf.kmeans_init(lists, 24)
    want, _ = ivf.ivf_knn(lists, C, 3, k)
    (idx, _), count = launches(lambda: ivf_knn(_dev(lists), _dev(C), 3, k))
    assert (count["knn_tile_half_lists"] > 0) == half and (count["knn_tile_half_other"] > 0) == half
    assert np.array_equal(idx.cpu().numpy(), want)
    # (the quantizer rounds its sums of this magnitude like any other)
    got = ivf_train(_dev(lists), 24, 2).cpu().numpy()
    assert np.abs(got - ivf.kmeans_train(lists, 24, 2)[0]).max() <= 1e-6 * np.abs(lists).max()


def test_later_passes_that_fail():
    """Lists of wide groups fill the first pass of 131,072 queries, lists of narrow ones the second: the third goes without half
    precision, and the second's queries are swept again."""
    from paper_1807_11824_amd import ivf_knn
    rng = np.random.default_rng(8)
    n, d, tau, k, nlist = 270_000, 72, 2, 20, 96
    narrow = np.arange(n) >= 131_500
    means = rng.standard_normal((16, d))
    X = (means[rng.integers(0, 8, n) + 8 * narrow] + np.where(narrow, 0.05, 1.0)[:, None] * rng.standard_normal((n, d))).astype(np.float32)
    C = np.concatenate([X[rng.choice(131_500, nlist // 2, replace=False)], X[131_500 + rng.choice(n - 131_500, nlist // 2, replace=False)]])
    name = rng.permutation(n)
    X = X[name]                             # (the lists are in the order of C whatever the rows')
    lists = ivf.ivf_lists(X, C)
    ends = np.cumsum([len(x) for x in lists])
    assert ends[nlist // 2 - 1] > 128_000
    (idx, d2), count = launches(lambda: ivf_knn(_dev(X), _dev(C), tau, k))
    chunks = -(-max(len(x) for x in lists) // 2048)
    assert count["knn_tile_half_lists"] == 2 * tau * chunks and count["knn_tile_mfma"] > tau * chunks
    rows = np.concatenate([rng.choice(l, 1) for l in lists if len(l)])
    want_idx, want_d2 = ivf.ivf_knn(X, C, tau, k, rows=rows)
    assert np.array_equal(idx[rows.tolist()].cpu().numpy(), want_idx)
    assert np.allclose(d2[rows.tolist()].cpu().numpy(), want_d2, rtol=1e-13, atol=1e-300)
