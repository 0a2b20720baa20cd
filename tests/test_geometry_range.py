"""Starts past a segment's sampled range (csrc/hpop_geom.h), on the CPU: one
that the scatter takes goes to the bucket in which a region query looks for
it, for bucket counts up to 2^24 and ranges up to 2^61 ns."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_scatter_and_query_agree_past_the_range(tmp_path):
    if not shutil.which("g++"):
        pytest.skip("no g++")
    exe = str(tmp_path / "geom_range")
    r = subprocess.run(["g++", "-std=c++17", "-O2", "-I", os.path.join(ROOT, "paper_2603_26576_amd", "csrc"),
                        os.path.join(ROOT, "tests", "native", "geom_range_main.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0, out.stdout + out.stderr
