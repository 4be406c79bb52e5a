"""The quantizer's farthest-point start (a training of no rounds) against the oracle, bit for bit: sixteen, thirty-two and all
lanes of a wave a sample row, columns that are no multiple of them, more workgroups than a wave looks through, ties."""
import numpy as np
import pytest

from oracle import ivf
from test_gpu_ivf import _dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,d,nlist", [
    (3, 1, 2), (40, 5, 1), (40, 5, 40), (700, 1, 64), (900, 15, 70), (3000, 16, 200), (3001, 17, 200), (5000, 63, 400), (5000, 65, 640),
    (2000, 127, 150), (2500, 255, 300), (2500, 256, 300), (2500, 257, 300), (1200, 511, 150), (900, 1024, 110), (900, 1025, 110),
    (70_000, 2, 2100),            # 16,800 sample rows: 263 workgroups of 64
    (4400, 1100, 530),            # 4240 sample rows: 265 workgroups of 16
    (9000, 258, 1100),            # 8800 sample rows: 275 workgroups of 32
])
def test_start(n, d, nlist):
    from paper_1807_11824_amd import ivf_train
    rng = np.random.default_rng(n + d)
    # small whole numbers (every sum is exact, many are equal), and real values in half of the cases
    X = rng.integers(-2, 3, (n, d)).astype(np.float32)
    if d % 2 == 0:
        X += rng.standard_normal((n, d)).astype(np.float32)
    if n > 100:
        X[n // 3: n // 2] = X[5]
    got = ivf_train(_dev(X), nlist, 0).cpu().numpy()
    assert np.array_equal(got, ivf.kmeans_init(X, nlist))
