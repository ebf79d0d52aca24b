"""The local join's products of fp32 rows: the distance tile against fp64, where a product formed in fewer bits, on another scale or in
another order would show."""
import numpy as np
import pytest
import torch

from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


def _tile(X, metric, shapes, seed=0):
    """Distances of blocks of those shapes and, fp64, per pair asked for: the product, the sum of the absolute products, how many products are
    not zero, the squared norms' sum and the norms' product."""
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
        Z = (P != 0).astype(np.float64)
        yield out[i][:a, :a + o][used], (P[:a] @ P.T)[used], (np.abs(P[:a]) @ np.abs(P).T)[used], (Z[:a] @ Z.T)[used], \
            np.add.outer((P[:a] ** 2).sum(1), (P ** 2).sum(1))[used], \
            np.multiply.outer(np.sqrt((P[:a] ** 2).sum(1)), np.sqrt((P ** 2).sum(1)))[used]


SHAPES = [(32, 32), (17, 30), (5, 0), (2, 0), (64, 64), (33, 95), (1, 127)]


def _points(kind, n, d, rng):
    X = rng.standard_normal((n, d))
    if kind == "scales":                       # norms over 24 orders of magnitude, values over six inside a row
        X *= np.exp(rng.normal(0, 2.3, (n, d)) + rng.uniform(-28, 28, (n, 1)))
    elif kind == "sparse":                     # about three values that are not zero
        X *= rng.random((n, d)) < 3.0 / d
    elif kind == "one large":                  # a value far above the others of its row, which no product of the others sees
        X[::2, 0] = 2.0 ** 20
        X[1::2, 0] = 0.0
    elif kind == "alike":                      # values that agree in all but their last bits
        X = 1.3717 + 1e-4 * X
    return X.astype(np.float32)


@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
@pytest.mark.parametrize("kind", ["scales", "sparse", "one large", "alike"])
@pytest.mark.parametrize("d", [1, 2, 3, 4, 7, 8, 16, 31, 32, 33, 64, 97, 128, 129, 250])
def test_products_are_those_of_fp32(d, kind, metric):
    """A sum of m products, each added to it in fp32, is within m 2^-24 of the sum of the absolute products (2^-24 for every rounding; products
    that are zero round nothing), whatever the rows' scales: the bound is per product and not per norm.  Norms are d + 4 such roundings
    of |x|^2 + |y|^2; the inner product has nothing else."""
    X = _points(kind, 500, d, np.random.default_rng(d))
    eps = 2.0 ** -24
    for got, gram, size, m, nsum, nmul in _tile(X, metric, SHAPES):
        if metric == "l2":
            want, tol = np.maximum(nsum - 2 * gram, 0), 2 * (m + 1) * eps * size + (d + 4) * eps * nsum
        elif metric == "ip":
            want, tol = -gram, (m + 1) * eps * size
        else:
            some = nmul > 0                    # (a row of zeros has no direction)
            got, gram, size, m, nmul = got[some], gram[some], size[some], m[some], nmul[some]
            want, tol = 1 - gram / nmul, (m + 1) * eps * size / nmul + (d + 8) * eps
        assert (np.abs(got - want) <= tol).all(), np.max(np.abs(got - want) / np.maximum(tol, 1e-300))


@pytest.mark.parametrize("metric", ["l2", "ip", "cosine"])
@pytest.mark.parametrize("f16", [0, 1])
@pytest.mark.parametrize("d", [5, 50, 64, 84, 96, 116, 128, 132, 200])
def test_a_pair_has_one_distance(d, f16, metric):
    """The same two real-valued rows get the same bits in a block of at most 64 members (a wave, registers) and in a larger one (a workgroup,
    LDS), whichever of them comes first, from fp32 rows and from those rounded to fp16: lists and thresholds must not depend on where a pair
    met, and the update of short lists finds the repeats of a candidate by their equal keys."""
    rng = np.random.default_rng(d)
    X = rng.standard_normal((300, d)).astype(np.float32)
    b = knn.Builder(torch.from_numpy(X).cuda(), knn.default_params(8, 4, metric=metric, join_f16=f16))
    order = rng.permutation(300)[:128].astype(np.int32)
    seen = {}
    for members, sizes in ((order, (64, 64)), (order[::-1].copy(), (64, 64)), (order[:64], (64, 0)), (order[:64][::-1].copy(), (64, 0)),
                           (order[16:64], (30, 18)), (order[32:96], (40, 24)), (order[20:110], (50, 40))):
        blk = np.zeros((1, 128), dtype=np.int32)
        blk[0, :len(members)] = members
        out = b.join_distances(torch.from_numpy(blk), torch.tensor([sizes], dtype=torch.int32)).cpu().numpy()[0]
        for i in range(sizes[0]):
            for j in range(i + 1, len(members)):
                pair = (min(members[i], members[j]), max(members[i], members[j]))
                assert seen.setdefault(pair, out[i, j]) == out[i, j]
    b.close()


@pytest.mark.parametrize("d", [20, 128, 132])
def test_more_blocks_than_workgroups(d):
    """5000 blocks in one call, so that every workgroup (2048 of them) walks several: the tiles are those of the same blocks in calls of at most
    2000, each of which has a workgroup to itself.  A block's member data must stay until all its waves have used them."""
    rng = np.random.default_rng(d)
    nb = 5000
    X = rng.standard_normal((3000, d)).astype(np.float32) * np.exp(rng.normal(0, 2, (3000, 1))).astype(np.float32)
    blk = np.argsort(rng.random((nb, 3000), dtype=np.float32), axis=1)[:, :128].astype(np.int32)
    new = rng.integers(1, 65, nb)
    sizes = np.stack([new, 128 - new], axis=1).astype(np.int32)
    sizes[::7] = [20, 30]                                                  # (of at most 64 members: a wave's for short rows)
    sizes[5::11] = [64, 64]
    b = knn.Builder(torch.from_numpy(X).cuda(), knn.default_params(8, 4))
    whole = b.join_distances(torch.from_numpy(blk), torch.from_numpy(sizes)).nan_to_num()
    for s in range(0, nb, 2000):
        part = b.join_distances(torch.from_numpy(blk[s:s + 2000]), torch.from_numpy(sizes[s:s + 2000])).nan_to_num()
        assert torch.equal(whole[s:s + 2000], part)
    b.close()


@pytest.mark.parametrize("d,most", [(1, 2896), (2, 2048), (32, 500), (33, 500), (128, 255)])
def test_whole_numbers_under_exact_sums_are_exact(d, most):
    """2 d most^2 <= 2^24: every fp32 sum over products or squares is exact, so a distance is
    the exact one rounded once (points on either side of the origin are up to 4 d most^2 apart: more than 24 bits)."""
    rng = np.random.default_rng(d)
    X = rng.integers(-most, most + 1, (400, d)).astype(np.float32)
    X[:40] = most - rng.integers(0, 2, (40, d))
    for got, gram, _, _, nsum, _ in _tile(X, "l2", [(40, 24), (64, 64), (16, 16), (1, 127)], seed=1):
        assert (got == (nsum - 2 * gram).astype(np.float32)).all()


@pytest.mark.parametrize("n,d,bytes_", [(1500, 24, False), (66_000, 16, False), (66_000, 16, True)])
def test_a_handle_starts_again_after_phase_2(n, d, bytes_):
    """Phase 2 writes its lists where phase 1 keeps edges and adjacency words: a second build on the same handle
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
