"""The spatial order at the sizes where the sort changes its tile (1024, 2048 and 4096 words and more), against the oracle."""
import pytest

from paper_1807_11824_amd import synth
from test_gpu_tree import _gpu_tree
import numpy as np
import oracle
from helpers import launches, random_symmetric_csr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [8192, 8193, 9217, 32768, 60000, 122880, 122881, 131072, 131073, 262144, 262145, 524288, 524289])
def test_order(n):
    Y = synth.clustered_embedding(n, n_clusters=40, seed=n)
    want = oracle.tree(Y, bits=22, leaf_cap=8)
    got = _gpu_tree(Y, 22, 8)
    assert np.array_equal(got["keys"].view(np.uint64), want["keys"])
    assert np.array_equal(got["perm"], want["perm"])
    assert got["m"] == want["m"]


@pytest.mark.parametrize("n,renumber,counted", [(122_880, False, True), (122_881, False, False), (131_072, True, True), (131_073, True, False)])
def test_which_sort(n, renumber, counted):
    """Counting up to 122,880 points in the caller's numbering and 131,072 renumbered ones; the keys are the oracle's."""
    import torch
    from paper_1807_11824_amd import Tsne
    Y = synth.clustered_embedding(n, n_clusters=40, seed=n)
    rp, col, val = random_symmetric_csr(n, 3, seed=n)
    ts = Tsne(n, max_nnz=len(col) if renumber else 0, graph_order_iters=4, morton_bits=22)
    dev = torch.device("cuda:0")
    ts.set_P(*[torch.from_numpy(a).to(dev) for a in (rp, col, val)])
    _, count = launches(lambda: ts.gradient(torch.from_numpy(Y).to(dev)))
    assert (count["rank_merge"] == 1) == counted and (count["radix_scatter"] > 0) != counted
    assert np.array_equal(ts.export_tree()["keys"].cpu().numpy().view(np.uint64), oracle.tree(Y, bits=22, leaf_cap=8)["keys"])
    ts.close()
