"""GPU checks of the running bound of the brute force's first pass: vectors
longer than the register-panel GEMM takes (and, beside them, of its own
lengths), with 127 tiles a workgroup where the launch has 64 of them, so that
values are dropped by the bound before the histogram is whole.  Small integers: every product sum is
exact, and the answers must be equal to the exhaustive ones."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,d", [(0, 257), (0, 40), (1, 270), (1, 256),
                                    (2, 520), (2, 512)])
@pytest.mark.parametrize("m,n,t,grid", [(1000, 130_001, 500, None),
                                        (1000, 130_001, 500, "64"),
                                        (130, 70_000, 1, "8"),
                                        (9000, 20_000, 3000, None)])
def test_answers_and_threshold(gpu, monkeypatch, prec, d, m, n, t, grid):
    import torch

    import paper_1506_03872_amd as mad
    if grid:
        monkeypatch.setenv("MAD_BF_GRID", grid)
    g = torch.Generator(device="cuda")
    g.manual_seed(d + m)

    def side(rows):
        return torch.randint(-3, 4, (rows, d), generator=g,
                             device="cuda").float()
    A, B = side(m), side(n)
    A[m // 3] *= 2.0  # a few vectors well above the others
    B[n // 5] *= 4.0
    screen = 0 if prec < 2 else 20 * t  # (fp8's certified bound keeps all)
    res, st = mad.bruteforce_topk(A, B, t, precision=prec, t_screen=screen)
    C = (A @ B.t()).abs().reshape(-1)
    if prec == 2:  # those re-ranked hold at least t pairs above tau
        got = res["c"].abs()
        assert float(got.min()) >= 0.96 * st["tau"]
        assert torch.equal(C[res["i"] * n + res["j"]], got)
        assert bool((got[:-1] >= got[1:]).all())
        return
    top = torch.topk(C, t).values
    cand = torch.nonzero(C >= top[-1]).reshape(-1)  # ascending keys
    order = torch.sort(C[cand], descending=True, stable=True).indices[:t]
    assert torch.equal(res["i"] * n + res["j"], cand[order])
    assert torch.equal(res["c"].abs(), C[cand[order]])
    if prec == 0 and m < 1024:  # every row in the first pass: the t-th |c|,
        # less a margin of 2e-4 of it, down to the edge of its bin (2^-5)
        assert 0.96 * float(top[-1]) <= st["tau"] <= float(top[-1])
