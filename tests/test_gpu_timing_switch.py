"""Stage timing switched on and off between computes: records that are built
already are not built again, and a rebuild takes every stage's time."""
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("events", [800, 9000], ids=["one kernel", "passes"])
def test_timing_switch_builds_nothing(events):
    tr = tg.make_trace(5, 2, 2, 2, events, events, regions="tiles", n_regions=3)
    want = oracle.compute(tr)
    s, keep = new_session(tr)

    def stages():
        return [n for n, _ in hp.hpop_session_stage_times(s)]

    try:
        assert_same(engine_results(s, tr), want)
        for _ in range(2):
            hp.hpop_session_enable_timing(s, True)
            assert_same(engine_results(s, tr), want, "timed, no build")
            assert stages() == ["region"]
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want, "timed build")
            full = stages()
            assert full[:2] == ["reset", "stats"] and "merge_wave" in full and full[-1] == "region"
            hp.hpop_session_enable_timing(s, False)
            assert_same(engine_results(s, tr), want, "no build")
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want, "build")
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want, "build again")
    finally:
        hp.hpop_session_destroy(s)
