"""The limit of the entry point without allocation: a call of one resource, one
record batch and very many regions that filled the scratch array before the
regions' accumulators held a slice count still fits, a larger one does not."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2603_26576_amd as hp
import tracegen as tg

pytestmark = pytest.mark.gpu

LIMIT = 256 << 20
PER_REGION = 48 + 176 + 72 + 32  # descriptor, tree, nine accumulators, one resource's state times


def call(n):
    """n regions [T0, T0 + 1 + i) over 100 records of 7 ns every 10 ns."""
    s = torch.arange(100, dtype=torch.int64).cuda() * 10 + tg.T0
    e = s + 7
    torch.cuda.synchronize()
    arr = (hp.hpop_event_chunk * 1)(hp.hpop_event_chunk(0, tg.DEV_KERNEL, s.data_ptr(), e.data_ptr(), 100))
    t0 = np.full(n, tg.T0, np.int64)
    t1 = t0 + 1 + np.arange(n)
    out = (hp.hpop_metric_tree * n)()
    p64 = ctypes.POINTER(ctypes.c_int64)
    st = hp.lib().hpop_metrics_compute_static(0, 1, arr, 1, t0.ctypes.data_as(p64), t1.ctypes.data_as(p64), n, 0, out, None)
    return st, out


@pytest.mark.parametrize("fits", [True, False])
def test_regions_up_to_the_limit(fits):
    # 64 KiB for the call's other tables, which take less than 8 KiB
    n = (LIMIT - (64 << 10)) // PER_REGION if fits else LIMIT // PER_REGION + 2000
    print("case: %d regions" % n, flush=True)
    st, out = call(n)
    if not fits:
        assert st == hp.HPOP_E_ARG
        return
    assert st == hp.HPOP_OK, hp.lib().hpop_last_error(None)
    for i in [0, 3, 6, 7, 9, 10, 456, 990, 996, 997, 1000, 5000, n // 2, n - 1]:
        t = i + 1  # ns into the records
        want = min(t // 10, 100) * 7 + (min(t % 10, 7) if t < 1000 else 0)
        assert out[i].E == t and out[i].sumK == want, (i, out[i].E, out[i].sumK)
