"""The bin counts through every order of the library's calls, on the CPU: g++ builds pm_api.cpp over
launchers that only track whether the counts are zero (host_bins_driver.cpp).  Runs with and without
checkpoints, building blocks in between, calls that fail half way and captures that are dropped."""
import subprocess

from host_model import build


def test_counts_are_zero_before_every_count(tmp_path):
    res = subprocess.run([build(tmp_path)], capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stdout.startswith("ok"), res.stdout + res.stderr
