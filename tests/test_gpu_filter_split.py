"""The prunings' products of rows split into two fp16 numbers per value, where splitting can go wrong: low parts that count in full,
candidates far larger or smaller than the node (which take the fp32 products), a node at the origin, columns that end within a step.
Whole numbers with squared norms of at most 2^23: bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


def _points(kind, n, d, rng):
    if kind == "low parts":                    # one value a row is beyond 2048: it needs its low part
        X = rng.integers(0, 12, (n, d))
        X[np.arange(n), rng.integers(0, min(d, 3), n)] = rng.integers(2048, 2850, n)
        return X
    if kind == "scales":                       # values of 0..3 next to multiples of 512 (beyond fp16 on the small nodes' scale), and zeros
        X = rng.integers(0, 4, (n, d))
        X[::3] *= int(np.sqrt(2 ** 23 / d)) // 3
        X[5::50] = 0
        return X
    return rng.integers(0, 40, (n, d))


@pytest.mark.parametrize("kind,n,d,k,hops", [
    ("low parts", 900, 66, 20, 1), ("low parts", 900, 68, 40, 1), ("low parts", 600, 70, 12, 2), ("low parts", 700, 129, 64, 1), ("low parts", 500, 1, 9, 1),
    ("scales", 900, 65, 20, 1), ("scales", 900, 68, 40, 1), ("scales", 500, 48, 10, 2), ("scales", 600, 100, 64, 1), ("scales", 500, 3, 12, 1),
    ("steps", 700, 31, 32, 1), ("steps", 700, 47, 33, 1), ("steps", 700, 48, 16, 1), ("steps", 700, 64, 24, 1), ("steps", 700, 65, 48, 1), ("steps", 700, 96, 49, 1),
    ("steps", 400, 97, 32, 1), ("steps", 400, 132, 8, 2)])
def test_split_products(kind, n, d, k, hops):
    rng = np.random.default_rng(n + d + k)
    X = _points(kind, n, d, rng).astype(np.float32)
    assert (X.astype(np.float64) ** 2).sum(1).max() <= 2 ** 23
    ids = np.stack([rng.choice(n, k, replace=False) for _ in range(n)]).astype(np.int32)      # (neighbours of every scale)
    Xg, ig = torch.from_numpy(X).cuda(), torch.from_numpy(ids).cuda()
    d_out = max(1, k // 2)
    for got, want in ((knn.prune_dist(Xg, ig, d_out, alpha=1.2, hops=hops), oracle.filter_dist(X, ids, hops, 64, 1.2, d_out)[0]),
                      (knn.prune_angle(Xg, ig, d_out, gamma_deg=60.0, hops=hops), oracle.filter_angle(X, ids, hops, 64, 60.0, d_out)[0]),
                      (knn.prune_dispersion(Xg, ig, d_out, hops=hops), oracle.filter_dpg(X, ids, hops, 64, d_out)[0])):
        assert (got.cpu().numpy() == want).all()


@pytest.mark.parametrize("power", [-55, -35, 20, 50])
def test_a_power_of_two_changes_nothing(power):
    """The angle rules multiply two squared lengths (of at most 2^17 here): with 4 power + 34 outside fp32's exponents the products are no
    longer the same numbers whatever forms the lengths, so they are asked at the two moderate powers only."""
    rng = np.random.default_rng(9)
    X = rng.integers(0, 40, (600, 80)).astype(np.float32)
    ids = torch.from_numpy(np.stack([rng.choice(600, 24, replace=False) for _ in range(600)]).astype(np.int32)).cuda()
    a, b = torch.from_numpy(X).cuda(), torch.from_numpy(X * np.float32(2.0 ** power)).cuda()
    assert torch.equal(knn.prune_dist(a, ids, 12), knn.prune_dist(b, ids, 12))
    if -40 < power < 24:
        assert torch.equal(knn.prune_angle(a, ids, 12), knn.prune_angle(b, ids, 12))
        assert torch.equal(knn.prune_dispersion(a, ids, 12), knn.prune_dispersion(b, ids, 12))
