"""The spatial order at the sizes where the sort changes its tile (1024, 2048 and 4096 words and more), against the oracle."""
import pytest

from paper_1807_11824_amd import synth
from test_gpu_tree import _gpu_tree
import numpy as np
import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8192, 8193, 9217, 32768, 60000, 131072, 131073, 262144, 262145, 524288, 524289])
def test_order(n):
    Y = synth.clustered_embedding(n, n_clusters=40, seed=n)
    want = oracle.tree(Y, bits=22, leaf_cap=8)
    got = _gpu_tree(Y, 22, 8)
    assert np.array_equal(got["keys"].view(np.uint64), want["keys"])
    assert np.array_equal(got["perm"], want["perm"])
    assert got["m"] == want["m"]
