"""Regions entered repeatedly, asked for again and again: every pass leaves the
intervals' accumulators clear for the next, with and without plain regions,
across rebuilds, new regions and new records."""
import ctypes

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import new_session

pytestmark = pytest.mark.gpu


def define_everywhere(s, R, parts):
    """A region that every resource enters at the same times: the sum of plain regions over `parts`."""
    n = len(parts) * R
    res = np.repeat(np.arange(R, dtype=np.int32), len(parts))
    a, b = (np.tile(np.array([p[i] for p in parts], np.int64), R) for i in (0, 1))
    out = ctypes.c_int32()
    assert hp.lib().hpop_region_define_multi(s, res.ctypes.data, a.ctypes.data, b.ctypes.data, n, ctypes.byref(out)) == hp.HPOP_OK


@pytest.mark.parametrize("plain", [0, 2])
def test_passes_repeat(plain):
    tr = tg.make_trace(11, 4, 4, 2, 2000, 600, regions="tiles", n_regions=9)
    parts = [r for r in tr.regions[1:9:2]]
    want = oracle.compute(tg.Trace(tr.n_hosts, tr.n_devices, tr.chunks, parts))["times"].sum(0)
    R = tr.n_hosts + tr.n_devices
    s, keep = new_session(tg.Trace(tr.n_hosts, tr.n_devices, tr.chunks, tr.regions[:plain]), device=True)
    try:
        define_everywhere(s, R, parts)
        for flags in (0, 0, hp.HPOP_FORCE_REBUILD, hp.HPOP_FORCE_REBUILD, 0):
            hp.hpop_metrics_compute_all(s, flags)
            got = np.array([hp.hpop_resource_times(s, plain, r) for r in range(R)])
            np.testing.assert_array_equal(got, want)
        define_everywhere(s, R, parts[:1])  # one more region: a new plan
        for _ in range(2):
            hp.hpop_metrics_compute_all(s)
            got = np.array([hp.hpop_resource_times(s, plain, r) for r in range(R)])
            np.testing.assert_array_equal(got, want)
    finally:
        hp.hpop_session_destroy(s)
