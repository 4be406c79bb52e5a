"""Sizes at which the launches of an iteration change: one workgroup builds the tree (up to 4096 points), the attraction
shares the walk's launch and the update adds Z up itself (up to 65,536).  Against the oracle, and one step against the
update rule applied to tsne_gradient's forces."""
import numpy as np
import pytest

import oracle
from helpers import grid_bits, random_symmetric_csr, rel_l2
from paper_1807_11824_amd import synth
from test_gpu_tree import _gpu_tree

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,leaf_cap", [(1023, 8), (1025, 8), (2049, 1), (3073, 16), (4095, 8), (4096, 5), (4096, 17), (4097, 8)])
def test_tree(n, leaf_cap):
    Y = synth.clustered_embedding(n, n_clusters=9, seed=n)
    Y[::7] = Y[0]
    want = oracle.tree(Y, bits=22, leaf_cap=leaf_cap)
    got = _gpu_tree(Y, 22, leaf_cap)
    assert got["m"] == want["m"] and np.array_equal(got["perm"], want["perm"])
    for key in ("depth", "lo", "hi", "leaf"):
        assert np.array_equal(got[key][:want["m"]].astype(np.int64), np.asarray(want[key]).astype(np.int64)), key
    side = float(np.ptp(Y, axis=0).max())
    assert np.abs(got["com"][:want["m"]] - want["com"]).max() <= 1e-6 * max(2 * side, 1e-30)


@pytest.mark.parametrize("n,renumber", [(2, False), (17, True), (4097, True), (65536, False), (65536, True), (65537, True)])
def test_forces_and_one_step(n, renumber):
    """Attraction and repulsion as in test_gpu_forces (1e-4); the step from the same forces in double: Y moves by
    lr gain grad, of which every operation is one rounding (1e-5 of the largest move)."""
    import torch
    from paper_1807_11824_amd import Tsne
    dev = torch.device("cuda:0")
    Y = synth.clustered_embedding(n, n_clusters=min(n, 20), seed=n)
    if n > 2:
        rp, col, val = random_symmetric_csr(n, min(20, n - 1), seed=n)
    else:
        rp, col, val = np.array([0, 1, 2], np.int32), np.array([1, 0], np.int32), np.array([0.5, 0.5], np.float32)
    ts = Tsne(n, max_nnz=len(col) if renumber else 0, graph_order_iters=8)
    ts.set_P(*[torch.from_numpy(a).to(dev) for a in (rp, col, val)])
    Yd = torch.from_numpy(Y).to(dev)
    A, R, Z = [t.cpu().numpy().astype(np.float64) for t in ts.gradient(Yd)]
    o = oracle.grad_bh(Y, rp, col, val.astype(np.float64), theta=0.5, leaf_cap=8, group=64, bits=grid_bits(n))
    assert rel_l2(A, o["A"]) <= 1e-4 and rel_l2(R, o["R"]) <= 1e-4 and abs(Z[0] - o["Z"]) <= 1e-5 * o["Z"]
    p = ts.params
    grad = 4.0 * (p.exaggeration * A - R / Z[0])
    move = -p.lr * np.where(grad == 0, p.gain_dec, 1.0 + p.gain_inc) * grad      # (velocity 0: the signs differ unless grad is 0)
    ts.step(Yd, 0)
    assert ts.status() == 0
    assert np.abs(Yd.cpu().numpy() - (Y + move)).max() <= 1e-5 * np.abs(move).max() + 2.0 ** -23 * np.abs(Y + move).max()
    ts.close()


@pytest.mark.parametrize("n,leaf_cap", [(1, 8), (700, 8), (4096, 1), (4096, 16)])
def test_counters_start_at_zero(n, leaf_cap, monkeypatch):
    """Every tree build zeroes the count of large cells and the sixteen counters of a resident walk.  With few points no walk
    of a whole chip is resident, so they are looked for in the workspace, which holds nothing but ones before: seventeen
    zero words and the padding behind them."""
    import torch
    from paper_1807_11824_amd import Tsne
    real = torch.empty
    monkeypatch.setattr(torch, "empty", lambda *a, **k: real(*a, **k).fill_(255) if k.get("dtype") == torch.uint8 else real(*a, **k))
    ts = Tsne(n, leaf_cap=leaf_cap)
    Y = torch.from_numpy(synth.clustered_embedding(n, n_clusters=min(n, 9), seed=n)).to("cuda:0")
    rp = torch.zeros(n + 1, dtype=torch.int32, device="cuda:0")
    ts.set_P(rp, torch.zeros(1, dtype=torch.int32, device="cuda:0")[:0], torch.zeros(1, device="cuda:0")[:0])
    ts.gradient(Y)
    words = ts.workspace[:ts.workspace.numel() // 256 * 256].cpu().numpy().view(np.int32).reshape(-1, 64)
    assert ((words[:, :17] == 0).all(axis=1) & (words[:, 17:] == -1).all(axis=1)).sum() == 1
    ts.close()


@pytest.mark.parametrize("renumber", [False, True])
def test_rows_in_the_walks_launch_are_the_same_to_the_bit(renumber):
    """65,536 points, whose rows of the attraction share the walk's launch, and one more point without entries, with which they
    have launches of their own: the same forces, bit for bit.  The last of the 65,536 points is the corner of the root square
    and the added one lies on it, so that nothing else moves in the order of the points (renumbered: along the embedding)."""
    import torch
    from helpers import launches
    from paper_1807_11824_amd import Tsne
    dev = torch.device("cuda:0")
    n = 65536
    Y = synth.clustered_embedding(n, n_clusters=20, seed=3)
    Y[-1] = Y.max(axis=0) + 1.0
    Y = np.concatenate([Y, Y[-1:]])
    rp, col, val = random_symmetric_csr(n, 40, seed=4)
    forces = []
    for m in (n, n + 1):
        ts = Tsne(m, max_nnz=len(col) if renumber else 0, graph_order_iters=0, reorder_every=1 if renumber else 0, far_tiles=1, morton_bits=22)
        ts.set_P(torch.from_numpy(np.concatenate([rp, rp[-1:]])[:m + 1].copy()).to(dev), torch.from_numpy(col).to(dev), torch.from_numpy(val).to(dev))
        if renumber:
            ts.step(torch.from_numpy(Y[:m].copy()).to(dev), 0)
        (A, _, _), count = launches(lambda: ts.gradient(torch.from_numpy(Y[:m].copy()).to(dev)))
        assert (count["bh_walk_rows"] == 1) == (m == n) and (count["attract_near" if renumber else "attract_csr"] == 1) == (m > n)
        if renumber:
            near, far = ts.P_layout()
            assert near > len(col) // 20 and far > len(col) // 20
        forces.append(A.cpu().numpy()[:n])
        ts.close()
    assert np.abs(forces[0]).max() > 0 and np.array_equal(forces[0], forces[1])
