"""The order that tsne_set_P derives from P does not depend on how the smoothing passes read P: by windows in LDS or by gathers,
with entries outside the window, or with so many that the passes are gathers again.  The same P is taken twice, once with
entries of value 0 at the ends of its rows, which change no sum (every lane adds them last) but the way the passes go."""
import numpy as np
import pytest

from helpers import launches

pytestmark = pytest.mark.gpu


def _graph(n, k, size, stray, seed):
    """CSR of n points in random numbering, k partners each in groups of `size` consecutive places, a share of them anywhere."""
    import scipy.sparse as sp
    rng = np.random.default_rng(seed)
    place = np.repeat(np.arange(n), k)
    other = np.minimum(place // size * size + rng.integers(0, size, len(place)), n - 1)
    far = rng.random(len(place)) < stray
    other[far] = rng.integers(0, n, int(far.sum()))
    name = rng.permutation(n)
    M = sp.coo_matrix((rng.random(len(place)) + 0.1, (name[place], name[other])), shape=(n, n)).tocsr()
    M = M + M.T
    M.setdiag(0); M.eliminate_zeros(); M.sort_indices()
    return M.indptr.astype(np.int32), M.indices.astype(np.int32), (M.data / M.sum()).astype(np.float32)


def _with_zeros(rp, col, val, extra, seed):
    """`extra` more entries at the end of every row, anywhere, of value 0."""
    n = len(rp) - 1
    rng = np.random.default_rng(seed)
    at = np.repeat(rp[1:], extra)
    return ((rp + extra * np.arange(n + 1)).astype(np.int32), np.insert(col, at, rng.integers(0, n, n * extra).astype(np.int32)),
            np.insert(val, at, np.zeros(n * extra, np.float32)))


def _orders(P, n, iters, after=None):
    """The permutations of the points that the context's workspace holds after set_P (the identity, the order, its inverse; where
    every row has far entries also the list of such rows, which has no order), and the launches of set_P.  after: a P that the
    context is given first."""
    import torch
    from paper_1807_11824_amd import Tsne
    dev = torch.device("cuda:0")
    t = Tsne(n, max_nnz=len(P[1]), graph_order_iters=iters)
    if after is not None:
        t.set_P(*[torch.from_numpy(a).to(dev) for a in after])
    P = [torch.from_numpy(a).to(dev) for a in P]
    _, count = launches(lambda: t.set_P(*P))
    words = t.workspace[:t.workspace.numel() // 256 * 256].view(torch.int32)
    starts = torch.arange(0, len(words) - n, 64, device=dev)
    ok = torch.ones(len(starts), dtype=torch.bool, device=dev)
    for power in (1, 2):                # (sums modulo 2^64)
        total = torch.cat([torch.zeros(1, dtype=torch.int64, device=dev), torch.cumsum(words.long() ** power, 0)])
        ok &= total[starts + n] - total[starts] == int((np.arange(n, dtype=np.int64) ** power).sum())
    found = {words[s: s + n].cpu().numpy().tobytes() for s in starts[ok].tolist()
             if torch.equal(torch.sort(words[s: s + n]).values, torch.arange(n, dtype=torch.int32, device=dev))}
    t.close()
    return found, count


@pytest.mark.parametrize("n,k,size,stray,extra,kernels", [
    (40_001, 24, 700, 0.05, 20, "gathers windows"),       # 48 entries a row and 68: gathers alone, windows of 38,912 alone
    (70_001, 36, 900, 0.01, 30, "both both"),             # under 2 % outside and far more
    (100_003, 36, 2000, 0.02, 12, "both both"),
    (150_001, 20, 2000, 0.05, 0, "gathers gathers"),      # short rows
    (270_001, 12, 1500, 0.0, 10, "both both"),            # short rows of many points: windows of 20,000
    (270_001, 40, 30_000, 0.0, 40, "both both"),          # shares of more rows, groups as wide as a window
])
def test_same_order(n, k, size, stray, extra, kernels):
    P = _graph(n, k, size, stray, seed=n)
    a, ca = _orders(P, n, 40)
    b, cb = _orders(_with_zeros(*P, extra, seed=k), n, 40)
    for c, want in zip((ca, cb), kernels.split()):
        # ten passes before the first copy are gathers in the caller's numbering, thirty are on a copy
        assert c["graph_relabel_k"] == 2 and c["graph_smooth_k"] == (10 if want == "windows" else 40)
        assert c["graph_smooth_window_k"] == (0 if want == "gathers" else 30)
        assert c["graph_sample_k"] == (2 if want == "both" else 0)
    assert len(a & b) == 3


@pytest.mark.parametrize("n,k", [(40_001, 48), (100_003, 48), (270_001, 12)])
def test_nothing_is_left_in_lds(n, k):
    """Windows are filled as far as entries reach; lanes past the end of a row read nothing else.  P of a context that was given
    values that are no numbers first (they fill every window) gives the order of a fresh one."""
    rp, col, val = _graph(n, k, 800, 0.0, seed=n)
    fresh, count = _orders((rp, col, val), n, 40)
    used, _ = _orders((rp, col, val), n, 40, after=(rp, col, np.full_like(val, np.nan)))
    assert count["graph_smooth_window_k"] == 30 and len(fresh & used) == 3
