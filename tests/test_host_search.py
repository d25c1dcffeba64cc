"""The group chain's search for a run start, on the CPU at the largest ranks a window may
have (2^31 - 2 samples): every position it reads lies inside the rank and the result is the
first length at or below the threshold.  Parity at the sizes a GPU test reaches is in
test_gpu_parity.py."""
import os
import subprocess

from paper_2606_19989_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


def test_run_start_search_at_the_largest_ranks(tmp_path):
    exe = str(tmp_path / "chain_search")
    r = subprocess.run([build.HIPCC, "--offload-host-only", "-O1", "-std=c++17", "-Wall", "-Werror", "-I", build.CSRC,
                        "-x", "hip", os.path.join(HERE, "host", "chain_search.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, (r.returncode, r.stdout)
