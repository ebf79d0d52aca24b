"""The pruning kernels at the sizes where the number of row groups (16 candidates each) and the collection of a
2-hop set change: bit for bit against the oracle on whole numbers, for the three rules."""
import numpy as np
import pytest
import torch

import oracle
from paper_2508_08744_amd import inputs, knn

pytestmark = pytest.mark.gpu


def _both(rule, X, ids, d_out, hops):
    Xg, Ig = torch.from_numpy(X).cuda(), torch.from_numpy(ids).cuda()
    if rule == "dist":
        want = oracle.filter_dist(X, ids, hops, 64, 1.1, d_out)
        got = knn.prune_dist(Xg, Ig, d_out, alpha=1.1, hops=hops, want_degrees=True)
    elif rule == "angle":
        want = oracle.filter_angle(X, ids, hops, 64, 60.0, d_out)
        got = knn.prune_angle(Xg, Ig, d_out, gamma_deg=60.0, hops=hops, want_degrees=True)
    else:
        want = oracle.filter_dpg(X, ids, hops, 64, d_out)
        got = knn.prune_dispersion(Xg, Ig, d_out, hops=hops, want_degrees=True)
    assert (got[0].cpu().numpy() == want[0]).all()
    assert (got[1].cpu().numpy() == want[1]).all()


@pytest.mark.parametrize("rule", ["dist", "angle", "dispersion"])
@pytest.mark.parametrize("k,d", [(32, 40), (33, 128), (40, 30), (47, 64), (48, 200), (49, 36)])
def test_one_hop_row_groups(rule, k, d):
    X = np.floor(inputs.make("C2", n=701, d=d, comps=7) / 4.0).astype(np.float32)
    ids, _ = oracle.brute_force_knn(X, k)
    ids = ids.astype(np.int32)
    ids[::5, k // 2] = -1                       # dead entries among the groups
    ids[::7, k - 1] = ids[::7, 0]
    _both(rule, X, ids, min(k, 40), 1)


@pytest.mark.parametrize("rule", ["dist", "angle", "dispersion"])
@pytest.mark.parametrize("k,n", [(32, 3001), (33, 6007), (64, 9001), (5, 40)])
def test_two_hops_of_random_rows(rule, k, n):
    # rows drawn at random: the second hop brings close to k * k distinct ids, the most the set has to hold
    # (few of them where n is small: most ids are met again)
    rng = np.random.default_rng(k)
    X = np.floor(inputs.make("C2", n=n, d=24, comps=5) / 4.0).astype(np.float32)
    ids = rng.integers(0, n, size=(n, k)).astype(np.int32)
    _both(rule, X, ids, min(k, 32), 2)


# the same where rows of X are no multiple of 16 bytes, which reads fewer rows of ids at a time: numbers of rows around what one step takes
@pytest.mark.parametrize("rule", ["dist", "angle", "dispersion"])
@pytest.mark.parametrize("k,n,d", [(32, 2003, 25), (33, 3001, 39), (9, 700, 30), (4, 60, 3)])
def test_two_hops_of_rows_read_value_by_value(rule, k, n, d):
    rng = np.random.default_rng(k + d)
    X = np.floor(inputs.make("C2", n=n, d=d, comps=5) / 4.0).astype(np.float32)
    ids = rng.integers(-1, n, size=(n, k)).astype(np.int32)
    _both(rule, X, ids, min(k, 32), 2)
