"""Builds redone for full slots, and builds with a start outside the sampled range
(which are not redone): new records answered once record no graph, and a forced
rebuild still replays one."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu

SPAN = 1 << 31


@pytest.mark.parametrize("why", ["range", "slots", "both"])
def test_redo_records_no_graph(why):
    rng = np.random.default_rng(len(why))
    n = 9000
    s = tg.T0 + SPAN // 4 + np.sort(rng.integers(0, SPAN // 2, size=n))
    if why != "range":
        s[: n // 2] = tg.T0 + SPAN // 2 + rng.integers(0, 100, size=n // 2)
        s.sort()
    if why != "slots":
        s[n // 2 if why == "range" else n - 1500] = tg.T0
    tr = tg.Trace(0, 1, [tg.Chunk(0, tg.DEV_KERNEL, s, s + rng.integers(0, SPAN // n, size=n))],
                  [(tg.T0, tg.T0 + SPAN), (tg.T0 + SPAN // 3, tg.T0 + SPAN // 2)])
    want = oracle.compute(tr)
    a, keep = new_session(tr, device=True)
    try:
        assert_same(engine_results(a, tr), want)
        assert hp.hpop_session_get_info(a).graph_replays == 0
        for i in range(1, 4):
            assert_same(engine_results(a, tr, hp.HPOP_FORCE_REBUILD), want)
            assert hp.hpop_session_get_info(a).graph_replays == i
    finally:
        hp.hpop_session_destroy(a)
