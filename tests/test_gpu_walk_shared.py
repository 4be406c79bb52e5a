"""The walk of a group by four waves (up to 65,536 points on 256 compute units) and by one (beyond), against the oracle."""
import numpy as np
import pytest

import oracle
from helpers import grid_bits, rel_l2
from paper_1807_11824_amd import synth
from test_gpu_forces import _gpu_forces

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,theta,leaf_cap,spread", [(300, 0.5, 1, 1.0), (3001, 0.0, 8, 1.0), (9000, 0.3, 20, 1e-3),
                                                     (20_000, 0.7, 1, 200.0), (65_536, 0.5, 8, 1.0), (65_537, 0.5, 8, 1.0)])
def test_forces(n, theta, leaf_cap, spread):
    """Clusters with 900 points on one spot (a large deepest leaf).  A force is a float sum, per wave, of the terms in
    the order they come, each addition off by at most half a unit of the sum so far: for some 700 list entries and the
    900 equal terms of the spot, which all err to one side, (700 + 900) 2^-24 = 1e-4 of the terms' sum.  Z leaves
    single precision after every batch of at most 512: 512 2^-24 / 2 = 1.5e-5."""
    Y = synth.clustered_embedding(n, n_clusters=12, seed=n) * np.float32(spread)
    Y[:: max(1, n // 900)] = Y[0]
    rp = np.zeros(n + 1, np.int32)
    _, R, Z, st = _gpu_forces(Y, rp, np.zeros(0, np.int32), np.zeros(0, np.float32), theta=theta, leaf_cap=leaf_cap)
    o = oracle.grad_bh(Y, rp, np.zeros(0, np.int32), np.zeros(0), theta=theta, leaf_cap=leaf_cap, group=64, bits=grid_bits(n))
    print("R", rel_l2(R, o["R"]), "Z", abs(Z - o["Z"]) / o["Z"], flush=True)
    assert st == 0 and rel_l2(R, o["R"]) <= 1e-4 and abs(Z - o["Z"]) <= 1.5e-5 * o["Z"]
