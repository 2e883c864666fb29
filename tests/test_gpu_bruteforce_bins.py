"""GPU checks of the brute force's threshold bins and of the size it gives
its survivor list, against the oracle's exhaustive answer.  All inputs are
small integers times powers of two, so every product sum is exact and the
answers must be equal."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def run(A, B, t, prec):
    import torch
    import paper_1506_03872_amd as mad
    res, st = mad.bruteforce_topk(torch.from_numpy(A).cuda(),
                                  torch.from_numpy(B).cuda(), t,
                                  precision=prec)
    n = B.shape[0]
    return (res["i"].cpu().numpy() * n + res["j"].cpu().numpy(),
            res["c"].cpu().numpy().astype(np.float64), st)


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("span", [0, 6, 30, 90])
def test_bins_over_the_exponent_range(gpu, prec, span):
    # row scales down to 2^-span: with t past the large rows, the t-th bound
    # lies in the fine bins (span 0, 6), in the coarse ones (30) or far below
    # both (90)
    g = np.random.default_rng(span)
    m, n, d, t = 260, 130, 24, 400
    A = g.integers(-8, 9, size=(m, d)).astype(np.float32)
    B = g.integers(-8, 9, size=(n, d)).astype(np.float32)
    A[2:] *= np.float32(2.0 ** -span)
    k, c, _ = run(A, B, t, prec)
    k_ex, c_ex = oracle.bruteforce_dense(A, B, t)
    assert np.array_equal(k, k_ex)
    assert np.array_equal(c, c_ex)


@pytest.mark.parametrize("prec", [0, 1, 2])
def test_a_bound_below_every_finer_bin(gpu, prec):
    # one huge pair of vectors, all others 2^-240 of their product: the t-th
    # bound lies below the certified filter's bins, and it takes those that
    # cover all floats
    g = np.random.default_rng(7)
    m, n, d, t = 140, 70, 12, 50
    A = g.integers(1, 9, size=(m, d)).astype(np.float32)
    B = g.integers(1, 9, size=(n, d)).astype(np.float32)
    A *= np.float32(2.0 ** -60)
    B *= np.float32(2.0 ** -60)
    A[0] *= np.float32(2.0 ** 120)
    B[0] *= np.float32(2.0 ** 120)
    # the huge vectors' products with the others are left out: disjoint halves
    A[0, d // 2:] = 0.0
    B[0, d // 2:] = 0.0
    A[1:, :d // 2] = 0.0
    B[1:, :d // 2] = 0.0
    k, c, _ = run(A, B, t, prec)
    k_ex, c_ex = oracle.bruteforce_dense(A, B, t)
    assert np.array_equal(k, k_ex)
    assert np.array_equal(c, c_ex)


@pytest.mark.parametrize("prec", [0, 1])
@pytest.mark.parametrize("sampled", [True, False])
def test_more_survivors_than_the_first_list(gpu, prec, sampled):
    # every |c| equal: all 2.2e6 pairs reach the threshold, more than the
    # default list of 2^20.  sampled: the subset of rows that sets the
    # threshold sees them; else its rows are zero and the list is grown
    # after the first run
    m, n, d, t = 1500, 1500, 16, 30
    A = np.ones((m, d), np.float32)
    if not sampled:
        A[::8] = 0.0
    B = np.ones((n, d), np.float32)
    k, c, st = run(A, B, t, prec)
    assert st["candidates"] > (1 << 20)
    rows = np.flatnonzero(A[:, 0])
    assert np.array_equal(k, rows[0] * n + np.arange(t))
    assert np.all(c == d)
