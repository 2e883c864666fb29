"""GPU parity of the MIPS batch's LDS-summed queries (units of 4096 samples
ordered by ranges of i, one table in LDS per range) at the edges of units,
bins and table sizes, beside queries whose budget keeps a table in memory
(above 2^18 samples).  Bar: every query's score table is the oracle's bit for
bit, with its candidate counts and its top t (as in test_gpu_mips.py)."""
import numpy as np
import pytest

import workloads
from test_gpu_mips import SEED, _check_query, _oracle_query, to_dev

pytestmark = pytest.mark.gpu


def check(A, Q, s, tp, t, chunk=None, prec=0):
    import paper_1506_03872_amd as mad
    s, tp = np.array(s, np.int64), np.array(tp, np.int64)
    gp = mad.MipsPlan.create(to_dev(A))
    if chunk:
        gp.set_config(chunk, 4, 512)
    if prec:
        gp.set_verify_precision(prec)
    res = gp.batch(to_dev(Q), s, tp, t, seed=SEED)
    st = gp.mips_stats(len(s))
    closed = distinct = 0
    for q in range(len(s)):
        o, ok, ox, cl = _oracle_query(A, Q[q], q, s[q], tp[q], t)
        closed += cl
        distinct += len(ok)
        gk, gx, F = gp.query_scores(q)
        assert F == o["F"]
        assert np.array_equal(gk, ok) and np.array_equal(gx, ox), q
        assert st["n_pos"][q] == o["n_pos"]
        assert st["n_cand"][q] == len(o["tp_key"])
        _check_query(A, q, Q[q], res[q], o, t)
    assert st["closed"] == closed and st["distinct"] == distinct
    gp.close()


@pytest.mark.parametrize("chunk", [256, 1024, 65536])
@pytest.mark.parametrize("m", [1, 2, 255, 257, 3000])
def test_units_and_bins(gpu, m, chunk):
    # budgets at the edges of a unit and of a bin count, t' that takes all
    # candidates (dot products with the bins) and t' that cuts
    t = min(m, 3)
    s = [1, 1023, 1024, 1025, 4095, 4096, 4097, 9000, 9000, 70000]
    tp = [10**6, 10**6, 5, 10**6, 10**6, 40, 10**6, 10**6, 7, 10**6]
    A, Q, _ = workloads.mips(m, 21, len(s), seed=m)
    check(A, Q, s, tp, t, chunk=chunk)


def test_tables_in_memory_beside_bins(gpu):
    # the largest budget summed in LDS, the smallest kept in memory, and
    # short queries, in one batch
    A, Q, _ = workloads.mips(5000, 12, 4, seed=1)
    check(A, Q, [1 << 18, (1 << 18) + 1, 600, 300000],
          [10**6, 10**6, 10, 50], 5)


@pytest.mark.parametrize("prec", [0, 1])
def test_a_bin_that_overflows_its_table(gpu, prec):
    # all the weight on the first 8192 rows of 60000, which are one bin of
    # eight at s = 8192: more distinct keys than the table has slots
    A, Q, _ = workloads.mips(60000, 16, 2, seed=5)
    A[8192:] *= 1e-6
    check(A, Q, [8192, 60000], [10**6, 10**6], 5, prec=prec)


@pytest.mark.parametrize("d", [513, 2049, 4096])
def test_the_widest_vectors(gpu, d):
    # stage-0 tables of up to 4096 slots beside a unit's samples in LDS
    A, Q, _ = workloads.mips(300, d, 3, seed=d)
    check(A, Q, [1000, 5000, 20000], [10**6, 10**6, 20], 3)
