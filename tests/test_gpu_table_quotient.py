"""GPU parity of the tables over the range of FP32 magnitudes: the builders
divide every prefix by its table's total through a reciprocal held once, and
the integer CDF has to be the IEEE division's for subnormal and huge weights,
for products of three of them (the stage-0 weights) and for totals whose
significand is all ones.  Bar: every table equal to the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def matrix(g, rows, d, lo, hi):
    x = np.ldexp(g.uniform(1.0, 2.0, (rows, d)),
                 g.integers(lo, hi, (rows, d))) * g.choice([-1, 1], (rows, d))
    return x.astype(np.float32)


# sizes at the edges of the builders: one wave (<= 512 slots, 1 to 8 a lane),
# the exact FP64 walk (up to 2^21 slots) and the stored quanta (long rows)
@pytest.mark.parametrize("m,n,d", [(64, 65, 33), (200, 511, 129),
                                   (600, 1025, 70), (70, 40, 1100)])
@pytest.mark.parametrize("lo,hi", [(-149, -120), (90, 110), (-60, 60),
                                   (-1, 0)])
def test_quotient(gpu, m, n, d, lo, hi):
    import torch

    import paper_1506_03872_amd as mad
    g = np.random.default_rng(m + lo + 200)
    if lo == -1:  # totals just below a power of two
        A = np.full((m, d), 1.0, np.float32)
        B = np.full((n, d), 1.0, np.float32)
        A[:, -1] = B[:, -1] = np.float32(1 - 2.0 ** -24)
        A[-1] = B[-1] = np.float32(1 - 2.0 ** -24)
    else:
        A, B = matrix(g, m, d, lo, hi), matrix(g, n, d, lo, hi)
    gp = mad.Plan.dense(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    op = oracle.Plan.dense(A, B)
    for which, seg in ([(0, 0)] + [(w, k) for w in (1, 2)
                                   for k in (0, 1, d // 2, d - 1)]
                       + [(3, i) for i in (0, m // 2, m - 1)]):
        got, want = gp.table(which, seg), op.table(which, seg)
        assert np.array_equal(got[0], want[0]), (which, seg)
        assert np.array_equal(got[1], want[1]), (which, seg)


# blocks of 4, 8 and 16 tables (from 4096 and 8192 tables on) of one to four
# runs of 128 items, the last block and the last run full and not
@pytest.mark.parametrize("m,d", [(4095, 128), (4100, 127), (8192, 129),
                                 (8205, 100), (8209, 8), (4099, 257),
                                 (4096, 512), (300, 385)])
def test_blocks_of_tables(gpu, m, d):
    import torch

    import paper_1506_03872_amd as mad
    g = np.random.default_rng(m + d)
    A = g.standard_normal((m, d)).astype(np.float32)
    A[m - 2] = 0.0  # a dead table
    B = g.standard_normal((7, d)).astype(np.float32)
    gp = mad.Plan.dense(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    op = oracle.Plan.dense(A, B)
    for i in (0, 1, 15, 16, m // 2, m - 17, m - 3, m - 2, m - 1):
        got, want = gp.table(3, i), op.table(3, i)
        assert np.array_equal(got[0], want[0]), i
        assert np.array_equal(got[1], want[1]), i


# tables of 1024 to 4096 slots (a workgroup each) and the sizes beside them,
# as columns of either side and as rows (whose stage 0 has the same length);
# runs full and not, dead tables, and a table of one item
@pytest.mark.parametrize("m,n,d", [(513, 1024, 9), (1025, 2048, 9),
                                   (2049, 4096, 9), (4095, 4097, 9),
                                   (640, 769, 65), (5, 7, 513), (5, 7, 1024),
                                   (5, 7, 2047), (5, 7, 4096), (5, 7, 4097)])
def test_mid_tables(gpu, m, n, d):
    import torch

    import paper_1506_03872_amd as mad
    g = np.random.default_rng(m + d)
    A = g.standard_normal((m, d)).astype(np.float32)
    B = g.standard_exponential((n, d)).astype(np.float32) ** 3
    A[:, 1] = 0.0  # a dead column
    A[2] = 0.0     # a dead row
    B[:, 2] = 0.0
    B[n // 2, 2] = -3.0  # one item
    gp = mad.Plan.dense(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    op = oracle.Plan.dense(A, B)
    for which, seg in ([(0, 0)] + [(w, k) for w in (1, 2)
                                   for k in (0, 1, 2, 3, d - 1)]
                       + [(3, i) for i in (0, 2, m - 1)]):
        got, want = gp.table(which, seg), op.table(which, seg)
        assert np.array_equal(got[0], want[0]), (which, seg)
        assert np.array_equal(got[1], want[1]), (which, seg)
    r = gp.topk(t=20, s=50_000, t_prime=200, seed=3)
    k, x, _ = gp.scores()
    assert len(k) and int(r["i"].max()) < m
