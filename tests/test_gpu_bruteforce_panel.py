"""GPU checks of the brute force's register-panel GEMM (fp32 and bf16 up to d
= 256, fp8 up to d = 512) at the edges of its steps, tiles and row panels, against
the oracle's exhaustive answer.  Inputs are small integers (exact in every
precision, and so are their sums), so the answers must be equal."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

# d at the edges of the 8-, 16- and 64-coordinate steps, of the change of tile
# width (fp32 128 | 129, bf16 64 | 65, fp8 128 | 129), of fp32's rows per wave
# (152 | 153) and even steps (160 | 161), and of the kernel's range (256 | 257,
# fp8 512 | 513); rows and columns at the edges of the 32- and 64-row waves,
# the 128- and 256-row panels and the 32- to 128-column tiles
SHAPES = [(1, 1, 1), (31, 33, 15), (64, 65, 16), (257, 127, 17),
          (255, 129, 63), (256, 128, 64), (513, 300, 65), (70, 1030, 100),
          (300, 257, 128), (300, 64, 129), (257, 131, 9), (258, 97, 152),
          (129, 161, 153), (127, 95, 160), (385, 33, 161), (511, 190, 241), (260, 255, 256),
          (130, 200, 257), (140, 190, 512), (140, 190, 513),
          # many work items per workgroup, and a sampled first pass
          (9000, 3001, 40)]


@pytest.mark.parametrize("prec", [0, 1, 2])
@pytest.mark.parametrize("shape", SHAPES)
def test_panel_edges(gpu, prec, shape):
    import torch
    import paper_1506_03872_amd as mad
    m, n, d = shape
    t = min(m * n, 60)
    g = np.random.default_rng([prec, m, n, d])
    A = g.integers(-8, 9, size=(m, d)).astype(np.float32)
    B = g.integers(-8, 9, size=(n, d)).astype(np.float32)
    a, b = torch.from_numpy(A).cuda(), torch.from_numpy(B).cuda()
    k_ex, c_ex = oracle.bruteforce_dense(A, B, t)
    for t_screen in (0, 4 * t):
        res, st = mad.bruteforce_topk(a, b, t, precision=prec,
                                      t_screen=t_screen)
        k = res["i"].cpu().numpy() * n + res["j"].cpu().numpy()
        c = res["c"].cpu().numpy().astype(np.float64)
        if t_screen == 0:
            assert np.array_equal(k, k_ex), st
        # screening: the computed values are exact here, so what it returns
        # is the head of the exact list; all of it when every row of A set
        # the threshold (fewer than 1024 rows)
        assert len(c) == t or (t_screen and m >= 1024)
        assert np.array_equal(c, c_ex[:len(c)]), st
