"""GPU check that the exact sparse answer's split weighs its heavy columns by
the GEMM that takes them: at 30,000 x 30,000 vectors over 2000 coordinates
the register-panel GEMM's 256 columns cost less than the next K step of the
longer one (1.70 against 2.12 ms in bf16), and a column of the fp8 filter no
less than one of the bf16 filter (2.55 against 3.01 ms)."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec", [1, 2])
def test_columns_of_the_panel_gemm(gpu, prec):
    import torch

    import paper_1506_03872_amd as mad
    m, d = 30_000, 2000
    a, b = (tuple(torch.from_numpy(np.ascontiguousarray(v)).cuda() for v in
                  workloads.powerlaw_csr(m, d, 24, seed=1, role=r))
            for r in (0, 1))
    res, st = mad.bruteforce_topk_csr(a, b, m, m, d, 1000, precision=prec)
    assert 64 <= st["heavy"] <= 256
    ref, _ = mad.bruteforce_topk_csr(a, b, m, m, d, 1000, precision=prec,
                                     heavy=320)
    for k in "ijc":
        assert torch.equal(res[k], ref[k])
