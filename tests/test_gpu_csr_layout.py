"""GPU parity of sparse plans at the edges of the table layout: table sizes
around each class (64, 128, 256, 512 items), above it (one to several runs
and 1024-slot blocks), empty tables, and more tables than one workgroup of
the layout takes (2048); plain and Gram plans (which share one transpose).
Bar: tables, and a run's candidates and pairs, equal to the oracle's."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# degrees of the first coordinates; the others hold at most one vector
DEGREES = [0, 1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513,
           1023, 1024, 1025, 2300]


def inputs(seed, rows, d):
    """CSR of `rows` vectors: coordinate k < len(DEGREES) in DEGREES[k] of
    them, and vector i holds coordinate len(DEGREES) + i % (d - ...)."""
    g = np.random.default_rng(seed)
    cols = [[] for _ in range(rows)]
    for k, n in enumerate(DEGREES):
        for i in g.choice(rows, size=n, replace=False):
            cols[i].append(k)
    nd = len(DEGREES)
    for i in range(1, rows):  # vector 0 keeps what it drew
        cols[i].append(nd + int(g.integers(d - nd - 1)))  # d - 1 unused
    ptr = np.zeros(rows + 1, np.int64)
    ptr[1:] = np.cumsum([len(c) for c in cols])
    idx = np.concatenate([np.sort(np.array(c, np.int32)) for c in cols])
    val = g.standard_normal(idx.size).astype(np.float32)
    return ptr, idx.astype(np.int32), val


def dev(x):
    import torch
    return tuple(torch.from_numpy(v).cuda() for v in x)


@pytest.mark.parametrize("gram", [False, True])
@pytest.mark.parametrize("d", [30, 5000])
def test_layout_edges(gpu, gram, d):
    import paper_1506_03872_amd as mad
    rows = 2500
    a = inputs(1, rows, d)
    b = a if gram else inputs(2, rows, d)
    da = dev(a)
    db = da if gram else dev(b)
    gp = mad.Plan.csr(da, db, rows, rows, d,
                      flags=mad.MAD_FLAG_GRAM if gram else 0)
    op = oracle.Plan.csr(*a, rows, *b, rows, d)
    for k in list(range(len(DEGREES))) + [d - 2, d - 1]:
        for which in (1, 2):
            gthr, _, gitem = gp.table(which, k)
            othr, _, _, _, _, _ = op.table(which, k)
            assert np.array_equal(gthr, othr), (which, k)
    s, tp, t = 200_000, 500, 20
    for rep in range(2):
        r = gp.topk(t, s, tp, seed=3)
        if gram:
            break
        o = op.topk(seed=3, s=s, t_prime=tp, t=t)
        key, x, _ = gp.candidates()
        assert np.array_equal(key, np.sort(o["tp_key"]))
        assert np.array_equal(r["i"].cpu().numpy() * rows +
                              r["j"].cpu().numpy(), o["key"])
        gp.refresh()  # laid out again, from a checked structure
    if gram:
        # the same X as a plain plan's, symmetrised off the diagonal
        pp = mad.Plan.csr(da, tuple(v.clone() for v in da), rows, rows, d)
        pp.topk(t, s, tp, seed=3)
        pk, px, _ = pp.scores()
        i, j = pk // rows, pk % rows
        keep = i != j
        want = {}
        for q, v in zip((np.minimum(i, j) * rows +
                         np.maximum(i, j))[keep].tolist(), px[keep].tolist()):
            want[q] = want.get(q, 0) + v
        gk, gx, _ = gp.scores()
        assert dict(zip(gk.tolist(), gx.tolist())) == want
        pp.close()
    gp.close()
    op.close()
