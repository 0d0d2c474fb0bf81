"""The protocol by which a compaction's tiles read each other's sums, on the CPU (its header holds no device code)."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_sums_of_an_earlier_launch_with_the_same_epoch_are_refused(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = tmp_path / "lookback_host"
    subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-Wno-unknown-pragmas", "-I",
                    os.path.join(ROOT, "paper_2505_12112_amd", "csrc"),
                    os.path.join(ROOT, "tests", "c_client", "lookback_host.cpp"), "-o", str(exe)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "lookback ok" in r.stdout, r.stdout + r.stderr
