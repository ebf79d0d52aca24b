"""The local join's products of rows split into two fp16 numbers per value: the distance tile against fp64, where splitting can go
wrong: a row's own scale, values far below its norm, steps of 32 columns, low parts that count in full."""
import numpy as np
import pytest
import torch

from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


def _tile(X, metric, shapes, seed=0):
    """Distances of blocks of those shapes and, fp64, their products, norms and which pairs were asked for."""
    rng = np.random.default_rng(seed)
    b = knn.Builder(torch.from_numpy(X).cuda(), knn.default_params(8, 4, metric=metric))
    blk = np.zeros((len(shapes), 128), dtype=np.int32)
    sizes = np.array(shapes, dtype=np.int32)
    for i, (a, o) in enumerate(shapes):
        blk[i, :a + o] = rng.choice(len(X), size=a + o, replace=False)
    out = b.join_distances(torch.from_numpy(blk), torch.from_numpy(sizes)).cpu().numpy().astype(np.float64)
    b.close()
    for i, (a, o) in enumerate(shapes):
        P = X[blk[i, :a + o]].astype(np.float64)
        used = np.triu(np.ones((a, a + o), dtype=bool), 1)
        yield out[i][:a, :a + o][used], (P[:a] @ P.T)[used], np.add.outer((P[:a] ** 2).sum(1), (P ** 2).sum(1))[used], \
            np.multiply.outer(np.sqrt((P[:a] ** 2).sum(1)), np.sqrt((P ** 2).sum(1)))[used]


@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
@pytest.mark.parametrize("d", [1, 7, 31, 32, 33, 64, 97, 128, 129, 250])
def test_rows_of_any_scale(d, metric):
    """Norms over 24 orders of magnitude, values over six inside a row.  With n sums rounded to 2^-24 (the fp16 instruction adds 32
    products a time: 3 d / 32 of them, plus up to 32 inside one), a product's value good to 2^-22 (its factors 2^-23 each) and 2^-22 left
    out, |error| <= (2^-21 + (3 d / 32 + 34) 2^-24) |x||y|, and d 2^-24 of |x|^2 + |y|^2 for the norms."""
    rng = np.random.default_rng(d)
    X = rng.standard_normal((500, d)) * np.exp(rng.normal(0, 2.3, (500, d)) + rng.uniform(-28, 28, (500, 1)))
    X = X.astype(np.float32)
    prod = 2.0 ** -21 + (3 * d / 32 + 34) * 2.0 ** -24
    for got, gram, nsum, nmul in _tile(X, metric, [(32, 32), (17, 30), (5, 0), (2, 0), (64, 64), (33, 95), (1, 127)]):
        if metric == "l2":
            want, tol = np.maximum(nsum - 2 * gram, 0), 2 * prod * nmul + (d + 4) * 2.0 ** -24 * nsum
        elif metric == "ip":
            want, tol = -gram, prod * nmul
        else:
            want, tol = 1 - gram / nmul, prod + (d + 8) * 2.0 ** -24
        assert (np.abs(got - want) <= tol).all(), np.max(np.abs(got - want) / tol)


@pytest.mark.parametrize("d,most", [(1, 2896), (2, 2048), (32, 500), (33, 500), (128, 255)])
def test_whole_numbers_under_exact_sums_are_exact(d, most):
    """2 d most^2 <= 2^24: every fp32 sum over products or squares is exact, low parts (d = 1: beyond 2048) and all, so a distance is
    the exact one rounded once (points on either side of the origin are up to 4 d most^2 apart: more than 24 bits)."""
    rng = np.random.default_rng(d)
    X = rng.integers(-most, most + 1, (400, d)).astype(np.float32)
    X[:40] = most - rng.integers(0, 2, (40, d))
    for got, gram, nsum, _ in _tile(X, "l2", [(40, 24), (64, 64), (16, 16), (1, 127)], seed=1):
        assert (got == (nsum - 2 * gram).astype(np.float32)).all()


@pytest.mark.parametrize("n,d,bytes_", [(1500, 24, False), (66_000, 16, False), (66_000, 16, True)])
def test_a_handle_starts_again_after_phase_2(n, d, bytes_):
    """Phase 2 writes its lists and its codes where phase 1 keeps edges, adjacency words and split rows: a second build on the same handle
    equals the first, and looking at blocks, adjacency and distances between rounds of phase 2 changes nothing."""
    rng = np.random.default_rng(n)
    X = rng.uniform(0, 255, (30, d))[rng.integers(0, 30, n)] + rng.normal(0, 9, (n, d))
    X = np.clip(np.rint(X), 0, 255).astype(np.float32) / (1 if bytes_ else 2)          # (sums of halves are as exact)
    b = knn.Builder(torch.from_numpy(X).cuda(), knn.default_params(12, 6, seed=5, it1=3, it2=3))
    blk = torch.from_numpy(rng.integers(0, n, (3, 128), dtype=np.int32))
    sizes = torch.tensor([[20, 30], [64, 64], [3, 9]], dtype=torch.int32)
    graphs, tiles = [], []
    for look in (False, True):
        b.init()
        tiles.append(b.join_distances(blk, sizes))
        for _ in range(3):
            b.phase1_round()
        b.begin_phase2()
        for _ in range(3):
            b.phase2_round()
            if look:
                b.sample_blocks()
                b.block_adjacency()
                tiles.append(b.join_distances(blk, sizes))
        graphs.append(b.finalize())
    b.close()
    assert all(torch.equal(x, y) for x, y in zip(*graphs))
    assert all(torch.equal(torch.nan_to_num(t), torch.nan_to_num(tiles[0])) for t in tiles)
