"""Host checks of the free list that keeps destroyed plans' memory: devices,
sizes, its bound, ageing, failed allocations and threads, with the runtime
replaced by one of two devices on the host (mem_pool_check.cpp)."""
import os
import subprocess

HERE = os.path.dirname(os.path.abspath(__file__))


def test_free_list(tmp_path):
    exe = str(tmp_path / "mem_pool_check")
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-pthread",
                    os.path.join(HERE, "mem_pool_check.cpp"), "-o", exe],
                   check=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stdout + r.stderr
