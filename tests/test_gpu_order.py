"""Late rounds take the nodes in an order that brings neighbours together (rows of at least 96 values, 8 M values in all): the graph is that
of the same points without four columns of zeros, bit for bit (every sum is exact): 92 values are too short for the order, and at 128, where
it is made too, rows take another join."""
import numpy as np
import pytest
import torch

from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


# lists shorter than what a step looks at; parts; no phase 2; no late round of phase 1; early stop; the workgroup join; bytes; n that is no
# multiple of anything
@pytest.mark.parametrize("n,d,k,scale,prm", [
    (87_383, 96, 3, 0.5, dict(it1=5, it2=2)), (87_400, 96, 16, 0.5, dict(it1=4, it2=0, parts=1)), (90_001, 96, 32, 0.5, dict(it1=4, it2=2, C=64)),
    (87_383, 96, 12, 0.5, dict(it1=2, it2=3, m=4)), (88_007, 96, 20, 1.0, dict(it1=5, it2=2, parts=4)), (88_007, 96, 10, 0.5, dict(it1=8, it2=8, delta=0.001)),
    (65_537, 132, 8, 0.5, dict(it1=5, it2=1)), (65_537, 132, 40, 1.0, dict(it1=4, it2=1)), (87_381, 99, 8, 0.5, dict(it1=5, it2=1))])
def test_order_changes_nothing(n, d, k, scale, prm):
    rng = np.random.default_rng(n + k)
    X = rng.integers(0, 120, (n // 500, d - 4))[rng.integers(0, n // 500, n)] + rng.integers(-6, 7, (n, d - 4))
    X = (np.clip(X, 0, 120) * scale).astype(np.float32)
    X[n // 3:n // 3 + 40] = X[7]                                  # equal points
    params = knn.default_params(k, 0, seed=3, **dict(dict(delta=0.0), **prm))
    wide = torch.zeros((n, d), device="cuda")
    wide[:, :d - 4] = torch.from_numpy(X)
    ids, dist, st = knn.knn_build_ex(wide, params)
    ids0, dist0, st0 = knn.knn_build_ex(torch.from_numpy(X).cuda(), params)
    assert torch.equal(ids, ids0) and torch.equal(dist, dist0)
    assert st["updates"] == st0["updates"] and st["join_pairs"] == st0["join_pairs"]
