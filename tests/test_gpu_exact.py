"""The screened exact k-NN at the edges of its samples, tiles and number ranges, against the brute-force oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08744_amd import inputs, knn

pytestmark = pytest.mark.gpu


def _check(X, k, metric, rows, static=False):
    Xg = torch.from_numpy(X).cuda()
    rg = torch.from_numpy(rows).cuda()
    ids, dist = (knn.exact_knn_static if static else knn.exact_knn)(Xg, k, metric, rg)
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy().astype(np.float64)
    mcode = knn.METRICS[metric]
    oi, od = oracle.brute_force_knn(X, k, mcode, rows)
    # An fp32 sum of d terms is off by at most (d + 4) half ulps of the sum of their magnitudes: the L2 distance itself,
    # |x| |y| for the products (1 for the cosine).  Where an id differs, the two true distances differ by no more than both errors.
    X64 = X.astype(np.float64)
    eps = (X.shape[1] + 4) * 2.0 ** -24
    nrm = np.sqrt((X64 ** 2).sum(1))
    size = {"l2": np.abs(od), "ip": nrm[rows][:, None] * nrm[oi], "cosine": np.full(od.shape, 4.0)}[metric]
    if metric == "ip":
        size = np.maximum(size, nrm[rows][:, None] * nrm[ids])
    assert (np.abs(dist - od) <= 2 * eps * size).all()
    for q, j in np.argwhere(ids != oi):
        a = oracle.distance(X, mcode, int(rows[q]), int(ids[q, j]))
        assert abs(a - od[q, j]) <= 2 * eps * size[q, j]
    assert (ids != rows[:, None]).all() and all(len(set(r)) == k for r in ids.tolist())


# rows around the size of the first sample and the next ones, queries around the tiles and the line between the two scans,
# rows of one 16-byte piece, of whole steps, of one value more
@pytest.mark.parametrize("n,d,k,nq,metric", [
    (65, 1, 64, 65, "l2"), (2047, 64, 33, 64, "l2"), (2048, 65, 1, 65, "ip"), (2049, 128, 64, 128, "cosine"), (4097, 32, 2, 63, "l2"),
    (8193, 33, 10, 129, "l2"), (8193, 129, 64, 257, "cosine"), (9000, 127, 17, 130, "ip"), (30000, 16, 32, 300, "l2"), (12000, 300, 5, 200, "l2")])
@pytest.mark.parametrize("whole", [True, False])
def test_exact_edges(n, d, k, nq, metric, whole):
    rng = np.random.default_rng(n + d)
    X = np.rint(rng.normal(0, 9, size=(n, d))).astype(np.float32) if whole else rng.normal(0, 1, size=(n, d)).astype(np.float32)
    if metric == "cosine":
        X[(X == 0).all(1)] = 1.0
    rows = rng.choice(n, size=nq, replace=False).astype(np.int64)
    _check(X, k, metric, rows)
    if d % 4 == 0:
        _check(X, k, metric, rows, static=True)


# values far from fp16's range, rows far from the origin, one row far from the others, masses of equal distances (more rows than a
# query's list has places: such queries are measured row by row)
@pytest.mark.parametrize("kind", ["tiny", "huge", "offset", "outlier", "twins"])
@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
def test_exact_number_ranges(kind, metric):
    rng = np.random.default_rng(5)
    n, d = 9001, 48
    X = rng.normal(0, 1, size=(n, d)).astype(np.float32)
    if kind == "tiny":
        X *= np.float32(1e-9)
    elif kind == "huge":
        X *= np.float32(1e7)
    elif kind == "offset":
        X += np.float32(500.0)
    elif kind == "outlier":
        X[17] *= np.float32(1e5)
    else:
        X = np.rint(X * 4).astype(np.float32)
        X[(X == 0).all(1)] = 1.0
        X[3000:8000] = X[2999]
    rows = np.concatenate([[17, 2999, 3000, 7999], rng.choice(n, size=150, replace=False)]).astype(np.int64)
    _check(X, 12, metric, rows)
    _check(X, 12, metric, rows[:40].copy(), static=True)


# rows without a defined distance (NaN, infinite) have no place in the order, but lists stay full and the defined rows in them are the
# nearest ones, wherever the others lie (in the first sample, too); every sum over whole numbers is exact
@pytest.mark.parametrize("n,nq,undefined", [(2049, 40, 3), (2049, 150, 3), (9001, 150, 5), (9001, 40, 8995), (150, 20, 4)])
@pytest.mark.parametrize("static", [False, True])
def test_exact_with_undefined_rows(n, nq, undefined, static):
    rng = np.random.default_rng(n + nq)
    k, d = 10, 64
    X = np.rint(rng.normal(0, 40, size=(n, d))).astype(np.float32)
    order = rng.permutation(n)
    good = np.sort(order[undefined:])
    X[order[:undefined], rng.integers(0, d, undefined)] = np.nan
    X[order[0]] = np.inf
    rows = good[rng.integers(0, len(good), nq)].astype(np.int64)
    Xg = torch.from_numpy(X).cuda()
    ids, dist = (knn.exact_knn_static if static else knn.exact_knn)(Xg, k, "l2", torch.from_numpy(rows).cuda())
    ids, dist = ids.cpu().numpy(), dist.cpu().numpy()
    m = min(k, len(good) - 1)
    oi, od = oracle.brute_force_knn(np.ascontiguousarray(X[good]), m, 0, np.searchsorted(good, rows).astype(np.int64))
    for q in range(nq):
        assert len(set(ids[q].tolist())) == k and (ids[q] >= 0).all()
        real = np.isin(ids[q], good)
        c = int(real.sum())
        assert (ids[q][real] == good[oi[q, :c]]).all() and (dist[q][real] == od[q, :c]).all()
        assert c >= min(m, k - undefined)
