"""GPU checks of the exact sparse brute force's split on the device: inputs
that it cuts, and those it hands to the host's rule (more pairs asked for
than there are products, equal degrees that no cut divides), against the
oracle's sparse FP64 product.  Values are small integers, so the products
are exact and the answers equal."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


def csr(rows):
    ptr = np.zeros(len(rows) + 1, np.int64)
    ptr[1:] = np.cumsum([len(r[0]) for r in rows])
    return (ptr, np.concatenate([r[0] for r in rows]).astype(np.int32),
            np.concatenate([r[1] for r in rows]).astype(np.float32))


def side(g, rows, d, hot, nnz):
    """Vectors with coordinate 0 (when hot) and nnz others, skewed to the
    front."""
    out = []
    for _ in range(rows):
        c = np.unique((d * g.random(nnz) ** 3).astype(np.int64))
        if hot:
            c = np.unique(np.append(c, 0))
        v = g.integers(1, 9, size=len(c)) * g.choice([-1, 1], size=len(c))
        out.append((c, v))
    return csr(out)


def run(a, b, m, n, d, t, heavy=0):
    import torch
    import paper_1506_03872_amd as mad
    dev = lambda x: tuple(torch.from_numpy(v).cuda() for v in x)
    res, st = mad.bruteforce_topk_csr(dev(a), dev(b), m, n, d, t,
                                      precision=1, heavy=heavy)
    return (res["i"].cpu().numpy() * n + res["j"].cpu().numpy(),
            res["c"].cpu().numpy().astype(np.float64), st)


@pytest.mark.parametrize("d", [3, 40, 2048, 2049, 9000])
@pytest.mark.parametrize("hot", [False, True])
def test_device_split(gpu, d, hot):
    g = np.random.default_rng([d, hot])
    m, n, t = 700, 500, 40
    a, b = side(g, m, d, hot, 12), side(g, n, d, hot, 9)
    k, c, st = run(a, b, m, n, d, t)
    k_ex, c_ex = oracle.exact_topk_sparse(a, b, m, n, d, t)
    assert np.array_equal(k, k_ex), st
    assert np.array_equal(c, c_ex)
    assert st["heavy"] >= 1


def test_fewer_products_than_asked(gpu):
    # three coordinates shared by few vectors: 11 pairs with a product,
    # t = 60.  The answer is the one of the host's rule.
    g = np.random.default_rng(5)
    m, n, d, t = 40, 30, 50, 60
    rows = [(np.array([i % 3]) if i < 6 else np.array([20 + i % 20]),
             g.integers(1, 9, size=1)) for i in range(m)]
    cols = [(np.array([j % 3]) if j < 5 else np.array([45]),
             g.integers(1, 9, size=1)) for j in range(n)]
    a, b = csr(rows), csr(cols)
    k, c, st = run(a, b, m, n, d, t)
    k1, c1, st1 = run(a, b, m, n, d, t, heavy=st["heavy"])
    assert np.array_equal(k, k1) and np.array_equal(c, c1)
    k_ex, c_ex = oracle.exact_topk_sparse(a, b, m, n, d, t)
    assert np.array_equal(k[:len(k_ex)], k_ex)
    assert np.array_equal(c[:len(k_ex)], c_ex)


def test_equal_degrees_that_no_cut_divides(gpu):
    # 5000 coordinates of equal degree: more than the 4096 that can be
    # heavy, in one bin; all of them light (few wedges) is not a cut with a
    # heavy coordinate either
    m = n = 5000
    d, t = 5000, 25
    g = np.random.default_rng(9)
    va, vb = g.permutation(d), g.permutation(d)
    a = csr([(np.sort([va[i], (va[i] + 1) % d]), g.integers(1, 99, size=2))
             for i in range(m)])
    b = csr([(np.sort([vb[j], (vb[j] + 2) % d]), g.integers(1, 99, size=2))
             for j in range(n)])
    k, c, _ = run(a, b, m, n, d, t)
    k_ex, c_ex = oracle.exact_topk_sparse(a, b, m, n, d, t)
    assert np.array_equal(k, k_ex)
    assert np.array_equal(c, c_ex)
