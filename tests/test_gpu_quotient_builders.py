"""GPU parity of the tables over the range of FP32 magnitudes, as in
test_gpu_table_quotient.py, in the builders that its sizes do not reach:
tables of more than 4096 items (the FP64 walks of a column's runs up to 2^21
items, the integer ones above, and the quanta of long rows), and sparse
tables of at most 64, 65 to 512 and more items.  Bar: every table equal to
the oracle's."""
import numpy as np
import pytest

import oracle
from test_gpu_csr_layout import DEGREES, dev, inputs
from test_gpu_table_quotient import matrix

pytestmark = pytest.mark.gpu

RANGES = [(-149, -120), (90, 110), (-60, 60), (-1, 0)]


def values(g, shape, lo, hi):
    if lo == -1:  # totals just below a power of two
        x = np.full(shape, 1.0, np.float32)
        x[-1] = np.float32(1 - 2.0 ** -24)
        return x
    if len(shape) == 1:
        return matrix(g, 1, shape[0], lo, hi)[0]
    return matrix(g, *shape, lo, hi)


@pytest.mark.parametrize("m,n,d", [(4097, 8193, 9), (70, 5000, 4100),
                                   (2_100_000, 5, 3)])
@pytest.mark.parametrize("lo,hi", RANGES)
def test_long_tables(gpu, m, n, d, lo, hi):
    import torch

    import paper_1506_03872_amd as mad
    g = np.random.default_rng(m + lo + 200)
    A, B = values(g, (m, d), lo, hi), values(g, (n, d), lo, hi)
    gp = mad.Plan.dense(torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda())
    op = oracle.Plan.dense(A, B)
    for which, seg in ([(0, 0)] + [(w, k) for w in (1, 2)
                                   for k in (0, d // 2, d - 1)]
                       + [(3, i) for i in (0, m // 2, m - 1)]):
        got, want = gp.table(which, seg), op.table(which, seg)
        assert np.array_equal(got[0], want[0]), (which, seg)
        assert np.array_equal(got[1], want[1]), (which, seg)
    gp.close()
    op.close()


@pytest.mark.parametrize("lo,hi", RANGES)
def test_sparse_tables(gpu, lo, hi):
    import paper_1506_03872_amd as mad
    rows, d = 2500, 30
    g = np.random.default_rng(lo + 200)
    a, b = ((x[0], x[1], values(g, x[2].shape, lo, hi))
            for x in (inputs(3, rows, d), inputs(4, rows, d)))
    gp = mad.Plan.csr(dev(a), dev(b), rows, rows, d)
    op = oracle.Plan.csr(*a, rows, *b, rows, d)
    for which, seg in ([(0, 0)] + [(w, k) for w in (1, 2)
                                   for k in range(len(DEGREES))]
                       + [(3, i) for i in (0, 1, rows // 2, rows - 1)]):
        got, want = gp.table(which, seg), op.table(which, seg)
        assert np.array_equal(got[0], want[0]), (which, seg)
    gp.close()
    op.close()
