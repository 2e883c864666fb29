"""GPU checks of the exact sparse brute force's bound on the light part: the
rounding of its fixed-point sums is bounded by the wedges that one pair can
have, so large values that form no wedge do not let more pairs through."""
import numpy as np
import pytest

import workloads
from test_gpu_bruteforce_csr import _check

pytestmark = pytest.mark.gpu


def with_entry(x, row, k, v):
    ptr, idx, val = x
    at = int(ptr[row + 1])  # the largest coordinate of its vector
    ptr = ptr.copy()
    ptr[row + 1:] += 1
    return (ptr, np.insert(idx, at, np.int32(k)),
            np.insert(val, at, np.float32(v)))


@pytest.mark.parametrize("heavy", [0, 64])
def test_large_values_without_wedges(gpu, heavy):
    import paper_1506_03872_amd as mad
    cfg, data = workloads.make("C3", seed=2, scale=0.003)
    a, b, m, n, d = data["a"], data["b"], data["m"], data["n"], cfg["d"]
    plain = _check(mad, a, b, m, n, d + 2, 100, prec=1, heavy=heavy)
    # one entry each on a coordinate that the other side does not have
    big = _check(mad, with_entry(a, m // 2, d, 2.0 ** 20),
                 with_entry(b, n // 3, d + 1, -2.0 ** 20), m, n, d + 2, 100,
                 prec=1, heavy=heavy)
    # (the two vectors themselves may pass with every partner: their light
    # norms carry the large values)
    assert big["light_candidates"] <= plain["light_candidates"] + m + n
    assert plain["light_candidates"] < plain["light_wedges"] // 10


def test_one_entry_per_vector(gpu):
    # no more than one wedge per pair, all of them light but one coordinate's
    import paper_1506_03872_amd as mad
    g = np.random.default_rng(6)
    m, n, d = 900, 700, 40

    def side(rows):
        return (np.arange(rows + 1, dtype=np.int64),
                g.integers(0, d, rows).astype(np.int32),
                g.standard_normal(rows).astype(np.float32))
    a, b = side(m), side(n)
    for heavy in (1, 0):
        _check(mad, a, b, m, n, d, 50, prec=0, heavy=heavy)
