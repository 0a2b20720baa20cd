"""Order of the region kernel's atomics in the code built for it: the slices of
a region add their sums and maxima, wait until the results are back, and only
then count themselves; the last one takes the accumulators after the count.
The kernel asks for the wait by hand (atomics of several lanes before one
lane's), so this reads it in the assembly."""
import os
import re
import subprocess

import pytest

from paper_2603_26576_amd import build as hbuild


def test_slices_wait_before_they_count(tmp_path):
    if not os.path.exists(hbuild.HIPCC):
        pytest.skip("no hipcc")
    out = str(tmp_path / "k.s")
    r = subprocess.run([hbuild.HIPCC] + hbuild.FLAGS + ["--cuda-device-only", "-S", os.path.join(hbuild.CSRC, "hpop_kernels.hip"),
                        "-o", out], capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr
    text = open(out).read()
    body = re.search(r"^_ZN4hpop8k_regionE\S*:(.*?)s_endpgm", text, re.S | re.M).group(1).splitlines()
    atomics = [(i, line.strip()) for i, line in enumerate(body) if "global_atomic" in line]
    wait = [i for i, line in enumerate(body) if "#ASMSTART" in line and body[i + 1].strip() == "s_waitcnt vmcnt(0)"]
    assert len(wait) == 1, wait
    before = [a.split()[0] for i, a in atomics if i < wait[0]]
    after = [a.split()[0] for i, a in atomics if i > wait[0]]
    # sums and maxima, each with its result asked for; then the count; then the last slice's reads
    assert sorted(before) == ["global_atomic_add_x2", "global_atomic_umax_x2"], atomics
    assert all(" sc0" in a for i, a in atomics if i < wait[0]), atomics
    assert after[0] == "global_atomic_add_x2" and after[1:] == ["global_atomic_swap_x2"] * 2, atomics
    count, reads = ([i for i, _ in atomics if i > wait[0]][k] for k in (0, 1))
    assert any("s_barrier" in line for line in body[count:reads])
