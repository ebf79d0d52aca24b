"""The prunings' products, where forming them in fewer bits or on another scale would show: values whose last bits count in full,
candidates far larger or smaller than the node, a node at the origin, columns that end within a step.
Whole numbers with squared norms of at most 2^23: bit for bit against the oracle; one real value a row: against fp32 arithmetic itself."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


def _points(kind, n, d, rng):
    if kind == "one large":                    # one value a row is beyond 2048
        X = rng.integers(0, 12, (n, d))
        X[np.arange(n), rng.integers(0, min(d, 3), n)] = rng.integers(2048, 2850, n)
        return X
    if kind == "scales":                       # values of 0..3 next to multiples of 512, and zeros
        X = rng.integers(0, 4, (n, d))
        X[::3] *= int(np.sqrt(2 ** 23 / d)) // 3
        X[5::50] = 0
        return X
    return rng.integers(0, 40, (n, d))


@pytest.mark.parametrize("kind,n,d,k,hops", [
    ("one large", 900, 66, 20, 1), ("one large", 900, 68, 40, 1), ("one large", 600, 70, 12, 2), ("one large", 700, 129, 64, 1), ("one large", 500, 1, 9, 1),
    ("scales", 900, 65, 20, 1), ("scales", 900, 68, 40, 1), ("scales", 500, 48, 10, 2), ("scales", 600, 100, 64, 1), ("scales", 500, 3, 12, 1),
    ("steps", 700, 31, 32, 1), ("steps", 700, 47, 33, 1), ("steps", 700, 48, 16, 1), ("steps", 700, 64, 24, 1), ("steps", 700, 65, 48, 1), ("steps", 700, 96, 49, 1),
    ("steps", 400, 97, 32, 1), ("steps", 400, 132, 8, 2)])
def test_products_of_whole_numbers(kind, n, d, k, hops):
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


def _rows_in_fp32(x, ids, alpha, d_out):
    """The distance rule over the neighbours where every row holds one value x[i] (its other columns are zero), every product, norm and
    difference rounded to fp32 once and nothing else rounded."""
    f = np.float32
    norm = x * x
    out = np.full((len(x), d_out), -1, dtype=np.int32)
    for p in range(len(x)):
        c = ids[p]
        diff = x[p] - x[c]
        dp = diff * diff
        order = np.lexsort((c, dp))
        c, dp = c[order], dp[order]
        rc = (norm[c][:, None] + norm[c][None, :]) - f(2) * (x[c][:, None] * x[c][None, :])
        thr = f(alpha) * f(alpha)
        kept = []
        for j in range(len(c)):
            if len(kept) < d_out and all(dp[j] < thr * rc[i, j] for i in kept):
                kept.append(j)
        out[p, :len(kept)] = c[kept]
    return out


@pytest.mark.parametrize("d,column", [(1, 0), (40, 3), (65, 64), (100, 17), (128, 0), (261, 260)])
def test_products_have_all_the_bits_of_fp32(d, column):
    """Neighbours at one part in 2^11 of their norms, so that the rule stands on the last bits of the products."""
    rng = np.random.default_rng(d)
    n, k = 500, 24
    x = (1.5 + 2.0 ** -11 * rng.standard_normal(n)).astype(np.float32)
    X = np.zeros((n, d), dtype=np.float32)
    X[:, column] = x
    ids = np.stack([rng.choice(np.delete(np.arange(n), p), k, replace=False) for p in range(n)]).astype(np.int32)
    for alpha in (1.0, 1.2):
        got = knn.prune_dist(torch.from_numpy(X).cuda(), torch.from_numpy(ids).cuda(), k, alpha=alpha)
        assert (got.cpu().numpy() == _rows_in_fp32(x, ids, alpha, k)).all()
