"""GPU checks of plans made from the memory of destroyed ones: results of
dense, sparse and MIPS plans of many sizes in sequence are those of plans
made from fresh memory, and mad_trim_memory gives back what is kept."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def calls():
    import torch

    import paper_1506_03872_amd as mad

    def dev(x):
        return torch.from_numpy(np.ascontiguousarray(x)).cuda()

    def dense(m, n, d, s):
        A, B = (dev(x) for x in workloads.dense_gaussian(m, n, d, seed=m))
        return lambda: mad.topk(A, B, t=10, s=s, t_prime=100, seed=4)

    def sparse(m, n, d, s):
        a, b = (tuple(dev(v) for v in workloads.powerlaw_csr(r, d, 8, seed=r))
                for r in (m, n))

        def run():
            p = mad.Plan.csr(a, b, m, n, d)
            r = p.topk(t=10, s=s, t_prime=100, seed=4)
            p.close()
            return r
        return run

    def mips(m, d, s):
        A, Q, _ = workloads.mips(m, d, 3, seed=m)
        A, Q = dev(A), dev(Q)

        def run():
            p = mad.MipsPlan.create(A)
            r = p.batch(Q, s, s, 5, seed=4)
            p.close()
            return {k: torch.cat([q[k] for q in r]) for k in r[0]}
        return run

    return [dense(300, 200, 16, 20_000), sparse(2000, 900, 300, 50_000),
            mips(5000, 24, [100, 5000, 300_000]), dense(2100, 5000, 40, 10**6),
            mips(300, 9, [64, 64, 64]), sparse(500, 4000, 5000, 10**5),
            dense(305, 199, 17, 20_100)]


def test_results_and_trim(gpu):
    import torch

    import paper_1506_03872_amd as mad
    fs = calls()
    fresh = []
    for f in fs:
        mad.trim_memory()
        fresh.append(f())
    mad.trim_memory()
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for order in (range(len(fs)), reversed(range(len(fs)))):
        for q in order:
            got = fs[q]()
            for k in fresh[q]:
                assert torch.equal(got[k], fresh[q][k]), (q, k)
    kept = mad.trim_memory()
    assert 0 < kept <= 2 << 30
    assert mad.trim_memory() == 0
    # all of it is the device's again (torch's own blocks of this test: less
    # than 64 MiB)
    assert torch.cuda.mem_get_info()[0] >= free0 - (64 << 20)


def test_threads_on_their_own_streams(gpu):
    # two threads make and destroy plans, each on a stream of its own, from
    # the one list
    import threading

    import torch

    import paper_1506_03872_amd as mad
    fs = [f for q, f in enumerate(calls()) if q not in (2, 4)]  # not MIPS
    mad.trim_memory()
    fresh = [f() for f in fs]
    torch.cuda.synchronize()
    wrong = []

    def work(order):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for q in order:
                got = fs[q]()
                for k in fresh[q]:
                    if not torch.equal(got[k], fresh[q][k]):
                        wrong.append((q, k))
            st.synchronize()
    n = len(fs)
    ts = [threading.Thread(target=work, args=([q % n for q in order],))
          for order in (range(3 * n), range(3 * n, 0, -1))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not wrong
    mad.trim_memory()
