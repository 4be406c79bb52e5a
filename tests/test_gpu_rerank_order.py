"""Re-rank of long rows (from 512 coordinates and 32 MB on) in the order of the nearest of the first 64 rows, against the oracle
(lists bit for bit): the labels say nothing, one block of query rows, two, a ragged last workgroup, no more rows than before."""
import numpy as np
import pytest

from helpers import launches
from test_gpu_build_p import _check_against_oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,same,k,ordered", [
    (17_000, 512, False, 30, 1),
    (17_155, 520, True, 1, 1),          # (the first 64 rows are one point)
    (66_001, 513, False, 20, 2),
    (66_001, 511, False, 20, 0),
    (16_000, 520, False, 20, 0),
])
def test_lists(n, d, same, k, ordered):
    rng = np.random.default_rng(n + d)
    X = 2.0 * rng.standard_normal((12, d))[rng.integers(0, 12, n)] + rng.standard_normal((n, d))
    if same:
        X[:64] = X[0]
    rows = np.unique(np.concatenate([np.arange(0, n, n // 20), [63, 64, n - 1]]))
    _, count = launches(lambda: _check_against_oracle(X.astype(np.float32), max(1.0, k / 3.0), k, rows=rows))
    assert count["rerank_sched_k"] == ordered and count["knn_tile_half"] > 0
