"""Steps recorded into HIP graphs: recorded and never replayed, replayed out of the order of their recording, and replayed
among eager calls.  Every result is the eager one, to the bit."""
import numpy as np
import pytest

from helpers import random_symmetric_csr
from paper_1807_11824_amd import synth

pytestmark = pytest.mark.gpu


# (rows in the caller's numbering with a launch of their own, with two streams and with one; sharing the walk's launch;
# one workgroup's tree; the renumbered copy)
@pytest.mark.parametrize("n,overlap,renumber", [(70_001, 1, False), (70_001, 0, False), (9001, 1, False), (3001, 1, True),
                                                (70_001, 1, True)])
def test_recorded_steps(n, overlap, renumber):
    import torch
    from paper_1807_11824_amd import Tsne
    dev = torch.device("cuda:0")
    rp, col, val = random_symmetric_csr(n, 12, seed=n)
    P = [torch.from_numpy(a).to(dev) for a in (rp, col, val)]
    Y0 = torch.from_numpy(synth.clustered_embedding(n, n_clusters=20, seed=n)).to(dev)
    kw = dict(overlap=overlap, max_nnz=len(col) if renumber else 0, graph_order_iters=8)
    s = torch.cuda.Stream()
    ref = Tsne(n, stream=s, **kw)
    # (a workspace that holds zeros: nothing in it is right by chance)
    zeros = torch.zeros_like(ref.workspace)
    del zeros
    t = Tsne(n, stream=s, **kw)
    torch.cuda.synchronize()
    with torch.cuda.stream(s):
        ref.set_P(*P); t.set_P(*P)
        if renumber:        # (the shares of the rows are settled by the first eager call with a new P)
            ref.gradient(Y0); t.gradient(Y0)
    Y = Y0.clone()
    torch.cuda.synchronize()
    graphs = []
    for it in (0, 300, 0):
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=s):
            t.step(Y, it)
        graphs.append(g)

    def eager_agrees():
        with torch.cuda.stream(s):
            a, b = t.gradient(Y0), ref.gradient(Y0)
        torch.cuda.synchronize()
        for x, y in zip(a, b):
            assert np.array_equal(x.cpu().numpy(), y.cpu().numpy())

    eager_agrees()
    Yr = Y0.clone()
    for which in (1, 2, 1, 0, 1, 0, 2):
        with torch.cuda.stream(s):
            graphs[which].replay()
            ref.step(Yr, (0, 300, 0)[which])
        torch.cuda.synchronize()
        assert np.array_equal(Y.cpu().numpy(), Yr.cpu().numpy())
        if which == 0:
            eager_agrees()
    with torch.cuda.stream(s):
        assert t.status() == 0
    t.close(); ref.close()
