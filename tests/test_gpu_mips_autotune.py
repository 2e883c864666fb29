"""GPU check that the MIPS autotuner tries only what can change a batch:
chunks above a unit (4096 samples) and table factors belong to queries of
more than 2^18 samples."""
import numpy as np
import pytest

import workloads
from test_gpu_mips import SEED, to_dev

pytestmark = pytest.mark.gpu


def test_trials_of_short_and_long_budgets(gpu):
    import paper_1506_03872_amd as mad
    A, Q, _ = workloads.mips(2000, 16, 6, seed=3)
    gp = mad.MipsPlan.create(to_dev(A))
    Qd = to_dev(Q)
    for s in ([200, 5000, 1000, 64, 9000, 1 << 18], [200] * 6):
        s = np.array(s, np.int64)
        for _ in range(3):
            gp.set_table_factor(8)
            c = gp.autotune(Qd, s, s, 5, seed=SEED, reps=1)
            # factors 2 and 4 are the tried ones: neither may be chosen
            assert c["slots"] == 8 and c["chunk"] in (1024, 4096)
    s = np.array([200, 5000, 1000, 64, 9000, 300_000], np.int64)
    c = gp.autotune(Qd, s, s, 5, seed=SEED, reps=1)
    assert c["slots"] in (2, 4, 8) and c["ms"] > 0
    gp.close()
