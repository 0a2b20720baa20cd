"""LDS layout of the kernel that takes the buckets the wave path hands over
(csrc/hpop_lds.h), on the CPU: no two waves of a workgroup share a byte,
whichever of their sorts each one runs."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_waves_share_no_lds(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    exe = str(tmp_path / "lds")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2603_26576_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "lds_main.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stdout + out.stderr
