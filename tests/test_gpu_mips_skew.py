"""GPU checks of MIPS batches on databases whose weight lies on few rows: the
LDS-summed queries' bins (the top bits of a hash of i) share it out wherever
it lies, and a bin that still holds more keys than its table is exact."""
import time

import numpy as np
import pytest

import workloads
from test_gpu_mips_bins import check

pytestmark = pytest.mark.gpu


def mips_bin(i, lb):
    """The kernels' bin of key i, one of 2^lb."""
    h = (i * 0x9E3779B1) & 0xFFFFFFFF
    h = ((h ^ (h >> 15)) * 0xB504F333) & 0xFFFFFFFF
    return h >> (32 - lb)


@pytest.mark.parametrize("prec", [0, 1])
def test_a_bin_with_more_keys_than_its_table(gpu, prec):
    # all the weight on the 4000 or so rows of one bin of 128 (the bins of a
    # query of 8192 samples), whose table has 2048 slots; the longer query
    # has it in four of 512 bins
    A, Q, _ = workloads.mips(520_000, 8, 2, seed=5)
    heavy = mips_bin(np.arange(len(A), dtype=np.uint64), 7) == 77
    assert 3500 < heavy.sum() < 4600
    A[~heavy] *= 1e-6
    check(A, Q, [8192, 60000], [10**6, 10**6], 5, prec=prec)


def test_time_on_rows_ordered_by_norm(gpu):
    # norms falling as i^-0.5: the same rows in random order take as long to
    # a few percent, where bins that are ranges of i took 4.9 times as long;
    # 2 leaves room for the clocks
    import torch

    import paper_1506_03872_amd as mad
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    m, d, nq, t = 1_000_000, 128, 4096, 10
    A = torch.randn(m, d, generator=g, device="cuda")
    A *= torch.arange(1, m + 1, device="cuda")[:, None] ** -0.5
    Q = torch.randn(nq, d, generator=g, device="cuda")
    s = np.round(10 ** np.random.default_rng(1).uniform(3, 5, nq))
    s = s.astype(np.int64)
    ms = []
    for rows in (A, A[torch.randperm(m, generator=g, device="cuda")]):
        gp = mad.MipsPlan.create(rows.contiguous())
        out = torch.zeros((nq * t, 3), dtype=torch.int64, device="cuda")
        n_out = torch.zeros(nq, dtype=torch.int64, device="cuda")
        best = 1e9
        for _ in range(6):  # the first plans the batch
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            gp.batch_raw(Q, s, s, t, 3, out, n_out)
            torch.cuda.synchronize()
            best = min(best, (time.perf_counter() - t0) * 1e3)
        ms.append(best)
        gp.close()
    print("ordered %.2f ms, shuffled %.2f ms" % tuple(ms), flush=True)
    assert ms[0] < 2 * ms[1]
