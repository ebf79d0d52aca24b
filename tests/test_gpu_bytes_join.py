"""The join on the 8-bit codes against the fp32 join: the same points halved are no whole numbers, and every fp32 sum over them
is exact all the same, so the two graphs agree bit for bit (distances of halved points times four)."""
import numpy as np
import pytest
import torch

from paper_2508_08744_amd import knn

pytestmark = pytest.mark.gpu


# sizes around the line between the joins and around column steps; signed values; the widest range and one beyond it;
# lists and samples that make blocks of up to 128 members; slots that collide often; every part count
@pytest.mark.parametrize("n,d,k,lo,hi,prm", [
    (65535, 20, 8, 0, 255, {}), (65536, 128, 32, 0, 255, {}), (65537, 1, 5, 0, 3, {}), (66001, 16, 16, -128, 127, dict(parts=1)),
    (66001, 17, 16, -300, -45, dict(parts=4)), (70003, 64, 20, 5, 260, dict(C=16)), (70003, 65, 20, 0, 256, {}), (70003, 127, 64, 0, 200, {}),
    (66001, 80, 33, 0, 255, dict(S=8, R=32, parts=8)), (66001, 96, 12, 0, 255, dict(R=0))])
def test_bytes_join_is_the_fp32_join(n, d, k, lo, hi, prm):
    rng = np.random.default_rng(n + d + k)
    centres = rng.uniform(lo, hi, size=(60, d))
    X = np.clip(np.rint(centres[rng.integers(0, 60, n)] + rng.normal(0, (hi - lo) / 12, size=(n, d))), lo, hi).astype(np.float32)
    X[0], X[1] = lo, hi
    X[n // 2:n // 2 + 3] = X[5]                                  # a few equal points
    params = knn.default_params(k, 0, seed=7, it1=3, it2=1, delta=0.0, **prm)
    Xg = torch.from_numpy(X).cuda()
    ids, dist, st = knn.knn_build_ex(Xg, params)
    idh, disth, sth = knn.knn_build_ex(Xg * 0.5, params)
    assert torch.equal(ids, idh) and torch.equal(dist, disth * 4.0)
    assert st["updates"] == sth["updates"] and st["join_pairs"] == sth["join_pairs"]
