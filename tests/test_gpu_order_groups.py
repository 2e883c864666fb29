"""The k order of more than 6.7e7 samples, whose counts are taken over groups
of several tiles: the scores of the ordered sampler equal those of the
unordered one (each sample is drawn once, whatever the order), for a last
group and a last tile that are not full, and for a last chunk of fewer
groups than the first."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("s", [70_000_001, 140_000_000, 68_000_000 + 4097])
def test_grouped_order(gpu, s):
    import torch

    import paper_1506_03872_amd as mad
    g = np.random.default_rng(s % 1000)
    A = torch.from_numpy(g.standard_normal((300, 40)).astype(np.float32))
    B = torch.from_numpy(g.standard_normal((200, 40)).astype(np.float32))
    got = []
    for order in (0, 1):
        p = mad.Plan.dense(A.cuda(), B.cuda())
        p.set_option(mad.MAD_OPT_SAMPLER_ORDER, order)
        if order and s == 140_000_000:  # 2^27 and the rest
            p.set_option(mad.MAD_OPT_ORDER_CHUNK, 1 << 27)
        p.topk(t=10, s=s, t_prime=100, seed=9)
        k, x, F = p.scores()
        at = np.argsort(np.asarray(k))
        got.append((np.asarray(k)[at], np.asarray(x)[at], F))
        del p
    assert got[0][2] == got[1][2]
    assert np.array_equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])
