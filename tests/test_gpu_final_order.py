"""GPU checks of the order of the returned pairs (|c| descending, then i, j)
at the sizes where the ranking kernel's rounds and workgroups end, with ties
in |c|.  Small integers: every product is exact."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t", [1, 15, 16, 17, 255, 256, 257, 1000, 2049])
def test_order_with_ties(gpu, t):
    import torch
    import paper_1506_03872_amd as mad
    g = np.random.default_rng(t)
    m, n, d = 70, 60, 6
    A = g.integers(-3, 4, size=(m, d)).astype(np.float32)
    B = g.integers(-3, 4, size=(n, d)).astype(np.float32)
    res, _ = mad.bruteforce_topk(torch.from_numpy(A).cuda(),
                                 torch.from_numpy(B).cuda(), t)
    k_ex, c_ex = oracle.bruteforce_dense(A, B, t)
    assert np.array_equal(res["i"].cpu().numpy() * n + res["j"].cpu().numpy(),
                          k_ex)
    assert np.array_equal(res["c"].cpu().numpy().astype(np.float64), c_ex)


def test_fewer_pairs_than_asked(gpu):
    # one sample, t = 40: at most one pair comes back (none when its
    # diamond is open or its score negative)
    import torch
    import paper_1506_03872_amd as mad
    g = np.random.default_rng(3)
    A = g.standard_normal((50, 8)).astype(np.float32)
    B = g.standard_normal((60, 8)).astype(np.float32)
    for seed in range(4):
        r = mad.topk(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda(),
                     40, 1, 40, seed=seed)
        o = oracle.Plan.dense(A, B).topk(seed=seed, s=1, t_prime=40, t=40)
        assert np.array_equal(r["i"].cpu().numpy() * 60 +
                              r["j"].cpu().numpy(), o["key"])
