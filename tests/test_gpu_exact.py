"""The screened exact k-NN at the edges of its samples, tiles and number ranges, against the brute-force oracle."""
import ctypes
import threading

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
    _compare(X, k, metric, rows, ids.cpu().numpy(), dist.cpu().numpy())


def _compare(X, k, metric, rows, ids, dist):
    dist = dist.astype(np.float64)
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


def _takes_f16(n, d, nq):
    """Whether tg_exact_knn screens such a search on rows rounded to fp16 (an internal function of the library)."""
    f = knn.lib()._Z16tg_exact_use_f16lil
    f.restype, f.argtypes = ctypes.c_bool, [ctypes.c_int64, ctypes.c_int, ctypes.c_int64]
    return f(n, (d + 3) // 4 * 4, nq)


def _check_f16(X, k, metric, rows, some):
    """All queries on fp16 rows against the fp32 rows, the first `some` of them against the oracle."""
    assert X.shape[1] % 4 == 0 and _takes_f16(*X.shape, len(rows))
    Xg, rg = torch.from_numpy(X).cuda(), torch.from_numpy(rows).cuda()
    got, want = knn.exact_knn(Xg, k, metric, rg), knn.exact_knn_static(Xg, k, metric, rg)
    # both measure what they list directly, in the same order of sums
    assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])
    _compare(X, k, metric, rows[:some], got[0][:some].cpu().numpy(), got[1][:some].cpu().numpy())


# (all of these are few enough pairs to be screened on the fp32 rows; the fp16 rows have tests of their own below)
# rows around the size of the first sample and the next ones, queries around the tiles,
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


def _ranged(rng, kind, n, d):
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
    return X


# values far from fp16's range, rows far from the origin, one row far from the others, masses of equal distances (more rows than a
# query's list has places: such queries are measured row by row)
@pytest.mark.parametrize("kind", ["tiny", "huge", "offset", "outlier", "twins"])
@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
def test_exact_number_ranges(kind, metric):
    rng = np.random.default_rng(5)
    n, d = 9001, 48
    X = _ranged(rng, kind, n, d)
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


# Rows whose squared norm is finite as it stands and infinite once scaled for fp16 (components of 2^57 where the others are at most 1), and
# rows without a norm: what shares a group of 16 rows of the scan with them still has its place in the lists.  The queries are exact in
# fp16, so their own residual is zero.  Every sum over the whole numbers (and over the powers of two) is exact.
@pytest.mark.parametrize("metric,kind", [("ip", "far"), ("l2", "far"), ("l2", "nan"), ("l2", "inf")])
def test_exact_f16_neighbours_of_rows_without_a_bound(metric, kind):
    n, d, k, nq = 40000, 128, 10, 500
    assert _takes_f16(n, d, nq)
    rng = np.random.default_rng(11)
    X = rng.integers(-1 if metric == "ip" else 0, 2, size=(n, d)).astype(np.float32)
    rows = rng.choice(np.arange(1000, n - 1000), size=nq, replace=False).astype(np.int64)
    check = np.arange(0, nq, 12)
    taken = set(rows.tolist()) | set(range(0, n, n // 512))          # queries, and the rows that the scale is taken from
    groups = 0
    for i, q in enumerate(check):
        g = 16 * int(rows[q] // 16 + 40)
        if taken & set(range(g, g + 16)) or (kind == "nan" and groups == 4):
            continue
        taken |= set(range(g, g + 16))
        groups += 1
        # three rows as near to the query as any, and one odd row, or nothing but odd rows behind them
        X[g:g + 3] = X[rows[q]]
        for r in range(g + 5, g + 16 if i % 2 and kind != "nan" else g + 6):
            X[r] = 2.0 ** 57 * (1 - 2 * rng.integers(0, 2, size=d)) if kind == "far" else np.nan if kind == "nan" else np.inf
    assert groups > 10 or kind == "nan"
    ids, dist = knn.exact_knn(torch.from_numpy(X).cuda(), k, metric, torch.from_numpy(rows).cuda())
    ids, dist = ids[torch.from_numpy(check).cuda()].cpu().numpy(), dist[torch.from_numpy(check).cuda()].cpu().numpy()
    good = np.nonzero(np.isfinite(X).all(1))[0]
    oi, od = oracle.brute_force_knn(np.ascontiguousarray(X[good]), k, knn.METRICS[metric], np.searchsorted(good, rows[check]).astype(np.int64))
    if kind != "nan":                                                # (an infinite distance comes last)
        assert (ids == good[oi]).all() and (dist == od).all()
        return
    for j in range(len(check)):                                      # a row without a distance may be listed anywhere: 4 of 10 places at most
        real = np.isin(ids[j], good)
        c = int(real.sum())
        assert c >= k - 4 and (ids[j][real] == good[oi[j, :c]]).all() and (dist[j][real] == od[j, :c]).all()


# The search on fp16 rows: every query against the search on fp32 rows (static, which never narrows), some against the oracle.  Rows of less than
# a step, of one to four whole steps, of one value more, queries too long to stay in LDS, queries that end within a tile, and 64, 128 and 256
# queries to a workgroup.
@pytest.mark.parametrize("n,d,k,nq,metric", [
    (140000, 16, 64, 1000, "l2"), (80000, 32, 1, 1000, "ip"), (60001, 36, 33, 999, "cosine"), (40000, 96, 10, 640, "l2"),
    (33001, 128, 32, 513, "ip"), (200003, 64, 20, 160, "l2"), (100001, 100, 3, 300, "ip"), (70001, 68, 50, 500, "cosine"), (33001, 132, 32, 513, "l2"), (20000, 300, 16, 400, "cosine"), (9001, 500, 5, 500, "ip"), (12000, 1200, 10, 150, "l2")])
@pytest.mark.parametrize("whole", [True, False])
def test_exact_f16_edges(n, d, k, nq, metric, whole):
    rng = np.random.default_rng(n + d)
    X = np.rint(rng.normal(0, 9, size=(n, d))).astype(np.float32) if whole else rng.normal(0, 1, size=(n, d)).astype(np.float32)
    if metric == "cosine":
        X[(X == 0).all(1)] = 1.0
    _check_f16(X, k, metric, rng.choice(n, size=nq, replace=False).astype(np.int64), 24)


# Tiles of 64 rows whose groups of 16 have norms (and residuals) of their own size get thresholds by the group, others one for the tile: one row far
# from the rest in every 64, in every 1000 (both kinds of tile), norms that grow from group to group, no two alike; one to four steps to a row,
# one, two and four waves side by side over the queries.
@pytest.mark.parametrize("n,d,k,nq,metric", [(140000, 28, 10, 900, "l2"), (200003, 64, 20, 160, "ip"), (70001, 96, 32, 300, "l2"), (50001, 128, 5, 500, "l2")])
@pytest.mark.parametrize("kind", ["one in 64", "one in 1000", "steps", "spread"])
def test_exact_f16_uneven_norms(n, d, k, nq, metric, kind):
    rng = np.random.default_rng(n + d)
    X = rng.normal(0, 1, size=(n, d)).astype(np.float32)
    if kind == "spread":
        X *= np.exp(rng.normal(0, 1, size=(n, 1))).astype(np.float32)
    elif kind == "steps":
        X *= (1 + np.arange(n) // 16 % 4)[:, None].astype(np.float32)
    else:
        X[11::64 if kind == "one in 64" else 1000] *= 100
    assert _takes_f16(n, d, nq)
    _check_f16(X, k, metric, rng.choice(n, size=nq, replace=False).astype(np.int64), 16)


@pytest.mark.parametrize("kind", ["tiny", "huge", "offset", "outlier", "twins"])
@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
def test_exact_f16_number_ranges(kind, metric):
    rng = np.random.default_rng(7)
    n, d = 45001, 48
    X = _ranged(rng, kind, n, d)
    rows = np.concatenate([[17, 2999, 3000, 7999], rng.choice(n, size=996, replace=False)]).astype(np.int64)
    _check_f16(X, 12, metric, rows, 40)


# Queries whose list overflows (3000 rows equal to them) are measured row by row by waves that are shared out among however many there
# are: none, one, a group of four and one more, all of them; on both kinds of rows, with slices of 256 rows and as many as fit.
@pytest.mark.parametrize("n,d,k,nq,f16", [(45001, 48, 64, 1000, True), (20000, 48, 33, 300, False), (6001, 32, 64, 61, False), (70000, 16, 1, 5, False)])
@pytest.mark.parametrize("listed", ["none", "one", "five", "all"])
def test_exact_overflowing_queries(n, d, k, nq, f16, listed):
    rng = np.random.default_rng(n + nq)
    X = rng.integers(0, 40, size=(n, d)).astype(np.float32)
    X[1000:4000] = X[1000] + 100.0                                   # (no other query's neighbours)
    m = {"none": 0, "one": 1, "five": 5, "all": nq}[listed]
    rows = rng.choice(np.arange(4000, n), size=nq, replace=False)
    rows[nq - m:] = 1000 + rng.permutation(3000)[:m]
    rows = rng.permutation(rows).astype(np.int64)
    assert _takes_f16(n, d, nq) == f16
    pick = np.concatenate([np.nonzero(rows < 4000)[0][:30], np.nonzero(rows >= 4000)[0][:30]])
    oi, od = oracle.brute_force_knn(X, k, 0, rows[pick])
    for f in (knn.exact_knn, knn.exact_knn_static):
        ids, dist = f(torch.from_numpy(X).cuda(), k, "l2", torch.from_numpy(rows).cuda())
        assert (ids.cpu().numpy()[pick] == oi).all() and (dist.cpu().numpy()[pick] == od).all()      # (every sum is exact)


def _pool_bytes_in_use():
    """Bytes that stream-ordered allocations of the default pool hold (hipMemPoolAttrUsedMemCurrent)."""
    hip = knn.lib()                                                  # (the runtime that the library is linked to)
    pool, used = ctypes.c_void_p(), ctypes.c_uint64()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), torch.cuda.current_device()) == 0
    assert hip.hipMemPoolGetAttribute(pool, 7, ctypes.byref(used)) == 0
    return used.value


def test_exact_scratch_is_taken_before_the_wait_and_given_back():
    """With row numbers the call waits for the stream.  The scratch is taken in front of that wait, where the last call's is still to be had, and given
    back whether the rows are good or not."""
    n, d, nq = 40000, 64, 1000
    X = torch.randn((n, d), device="cuda", generator=torch.Generator(device="cuda").manual_seed(1))
    rows = torch.arange(nq, device="cuda")
    want = knn.exact_knn(X, 8, "l2", rows)
    torch.cuda.synchronize()
    before = _pool_bytes_in_use()
    side = torch.cuda.Stream()
    got = []

    def call():
        with torch.cuda.stream(side):
            got.append(knn.exact_knn(X, 8, "l2", rows))

    with torch.cuda.stream(side):
        torch.cuda._sleep(400_000_000)                               # the call waits for this one
    worker = threading.Thread(target=call)
    worker.start()
    held = 0
    while not side.query() and held == 0:
        held = _pool_bytes_in_use() - before
    worker.join()
    torch.cuda.synchronize()
    assert held > n * d * 2                                          # (at least the fp16 copy of X)
    assert all(torch.equal(a, b) for a, b in zip(got[0], want))
    rows[nq - 1] = n
    for _ in range(3):
        with pytest.raises(knn.TagoreError, match="row %d out of range" % n):
            knn.exact_knn(X, 8, "l2", rows)
    torch.cuda.synchronize()
    assert _pool_bytes_in_use() == before
