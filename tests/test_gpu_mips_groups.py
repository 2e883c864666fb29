"""GPU checks of MIPS batches whose samples far outnumber what their score
tables would hold: the words of the LDS-summed queries are in memory a group
of queries at a time.  Bar: the score tables of queries on both sides of the
groups' borders are the oracle's bit for bit, as are their top t, and the
batch takes memory by the tables it replaces, not by its samples."""
import numpy as np
import pytest

import workloads
from test_gpu_mips import SEED, _check_query, _oracle_query, to_dev

pytestmark = pytest.mark.gpu


def run(m, d, s, tp, t, checked, limit):
    import torch

    import paper_1506_03872_amd as mad
    A, Q, _ = workloads.mips(m, d, len(s), seed=m)
    gp = mad.MipsPlan.create(to_dev(A))
    Qd = to_dev(Q)
    out = torch.zeros((len(s) * t, 3), dtype=torch.int64, device="cuda")
    n_out = torch.zeros(len(s), dtype=torch.int64, device="cuda")
    mad.trim_memory()
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    for seed in (SEED + 1, SEED):  # the second replays the layout
        gp.batch_raw(Qd, s, tp, t, seed, out, n_out)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] < limit
    cnt = n_out.cpu().tolist()
    for q in checked:
        o, ok, ox, _ = _oracle_query(A, Q[q], q, s[q], tp[q], t)
        gk, gx, F = gp.query_scores(q)
        assert F == o["F"]
        assert np.array_equal(gk, ok) and np.array_equal(gx, ox), q
        res = mad.unpack_pairs(out[q * t:(q + 1) * t], cnt[q])
        _check_query(A, q, Q[q], res, o, t)
    gp.close()


def test_many_samples_on_few_vectors(gpu):
    # 32769 queries of up to 2^18 samples on 1024 vectors: 69 GB of words and
    # 2^24 (query, bin) pairs in all; tables of 16 KB a query; other budgets
    # among them
    nq = 32769
    s = np.full(nq, 1 << 18, np.int64)
    s[[3, 700]] = [0, (1 << 18) + 1]
    s[[1, 5, 40]] = [70, 4097, 9000]
    run(1024, 4, s, np.where(s > 10**5, 10, s + 3), 3,
        [0, 1, 5, 40, 700, 127, 128, 255, 256, 257, 20000, nq - 1], 4 << 30)


def test_many_items(gpu):
    # 4200 queries of 256 bins or more: over 2^20 (query, bin) pairs while
    # the words are no more than the tables would be
    nq = 4200
    s = np.full(nq, 1 << 18, np.int64)
    run(261120, 4, s, np.full(nq, 20, np.int64), 3,
        [0, 2055, 2056, 4095, 4096, nq - 1], 40 << 30)
