"""Lists are sorted by networks on 32-bit keys, looked over and put right: whole builds on points whose distances are few (whole numbers of
a small range, so most neighbours in a list stand at equal distances and ids decide), against the oracle, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


# lists on either side of the two kinds of list update (32 entries), a list and its candidates in one network or in several batches (C slots
# a node), arrivals of one class only or of both; values per dimension: 2 (nearly everything equal) to 200 (pairs and threes)
@pytest.mark.parametrize("n,d,k,values,kw", [
    (900, 3, 32, 2, dict()), (1500, 8, 31, 3, dict(C=64)), (1500, 4, 33, 6, dict(parts=1)), (1200, 12, 10, 4, dict(C=256, parts=4)),
    (2000, 6, 17, 40, dict(C=32)), (2500, 16, 24, 200, dict()), (700, 2, 64, 30, dict())])
def test_builds_of_equal_distances(n, d, k, values, kw):
    rng = np.random.default_rng(n + d)
    X = rng.integers(0, values, size=(n, d)).astype(np.float32)
    prm = knn.default_params(k, 6, seed=5, **kw)
    ids, dist, _ = knn.knn_build_ex(torch.from_numpy(X).cuda(), prm)
    o = oracle.NNDescent(X, k, **oracle.device_model(prm))
    o.run(prm.it1, prm.it2)
    oi, od, _ = o.graph()
    assert (ids.cpu().numpy() == oi).all() and (dist.cpu().numpy().astype(np.float64) == od).all()
