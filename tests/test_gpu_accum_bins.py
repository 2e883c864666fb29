"""GPU checks of the score accumulation where its paths change: bins at the
edge of the one-round reduction (768 pairs in the 1024-slot table), with all
keys distinct, all equal or none; sizes at the edge of the wide tiles (2^24
pairs); and two splits after the first partition, which only more than
3.4e8 pairs take by themselves (smaller bins are asked for in a process of
its own, as the setting is read once).  Every key's sum is compared with a
numpy group-by, bit for bit."""
import os
import subprocess
import sys

import numpy as np
import pytest

from test_gpu_accumulate import EMPTY, mix64, run

pytestmark = pytest.mark.gpu

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def mad_gpu(gpu):
    import paper_1506_03872_amd as mad
    mad.lib()
    return mad


def test_reduction_edges(mad_gpu):
    # n = 16384 pairs: 32 bins by the top 5 hash bits
    g = np.random.default_rng(11)
    n = 16384
    cand = np.unique(g.integers(0, 1 << 40, 200_000, dtype=np.int64))
    b = mix64(cand.astype(np.uint64)) >> np.uint64(59)
    of = [cand[b == k] for k in range(32)]
    parts = [of[0][:768], of[1][:769],               # distinct
             g.choice(of[2][:300], 768), g.choice(of[3][:300], 769),
             np.full(768, of[4][0]), np.full(769, of[5][0]),
             of[6][:1], np.concatenate([of[7][:700], of[7][:68]])]
    k = np.concatenate(parts)
    rest = g.choice(np.concatenate(of[9:]), n - len(k))  # bin 8: no pair
    keys = np.concatenate([k, rest])
    g.shuffle(keys)
    assert len(keys) == n
    # increments on both sides of 2^51 at F = 50 (the two conversions)
    vals = (g.standard_normal(n) * 2).astype(np.float32)
    for F in (0, 20, 50):
        run(mad_gpu, keys, vals, F)


@pytest.mark.parametrize("extra", [-1, 0, 8191, 8193])
def test_wide_tiles(mad_gpu, extra):
    g = np.random.default_rng(12)
    n = (1 << 24) + extra
    keys = g.integers(0, 8_000_000_000, n, dtype=np.int64)
    keys[: n // 4] = g.integers(0, 1_000_000, n // 4)
    keys[g.random(n) < 0.1] = EMPTY
    vals = g.standard_normal(n).astype(np.float32)
    run(mad_gpu, keys, vals, 26)


CHILD = """
import sys
sys.path[:0] = [%r, %r]
import numpy as np
import paper_1506_03872_amd as mad
from test_gpu_accumulate import EMPTY, run
g = np.random.default_rng(13)
n = 36_000_000  # 256 pairs a bin: 18 bits, 10 of them in two splits
keys = g.integers(0, 40_000_000_000, n, dtype=np.int64)
keys[: n // 4] = g.integers(0, 3_000_000, n // 4)
keys[g.random(n) < 0.15] = EMPTY
print(run(mad, keys, g.standard_normal(n).astype(np.float32), 28))
"""


def test_two_splits(gpu):
    env = dict(os.environ, MAD_ACC_TARGET="256")
    r = subprocess.run([sys.executable, "-c",
                        CHILD % (os.path.dirname(HERE), HERE)], env=env,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0, r.stderr[-3000:]
