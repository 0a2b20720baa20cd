"""The tuning a session reports is the one its build takes: set back, it builds
the same buckets and answers."""
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("events,want", [(0, (320, 512)), (10_000, (320, 512)), (40_000, (320, 2048))])
def test_reported_tuning_set_back(events, want):
    tr = tg.make_trace(6, 2, 2, 2, events, events, regions="tiles", n_regions=3) if events else \
        tg.Trace(2, 2, [], [(0, 10)])
    ref = oracle.compute(tr)
    s, keep = new_session(tr)
    try:
        assert_same(engine_results(s, tr), ref)
        before = hp.hpop_session_get_info(s).n_buckets
        t = hp.hpop_session_get_tuning(s)
        assert (t.bucket_target, t.tile_elems, t.bucket_cap, t.scatter_slots) == want + (2048, 2048)
        hp.hpop_session_set_tuning(s, t.bucket_target, t.bucket_cap, t.tile_elems, t.scatter_slots)
        assert_same(engine_results(s, tr), ref, "set back")
        assert hp.hpop_session_get_info(s).n_buckets == before
        u = hp.hpop_session_get_tuning(s)
        assert bytes(u) == bytes(t)
        # a value asked for stays
        hp.hpop_session_set_tuning(s, tile_elems=4096)
        assert hp.hpop_session_get_tuning(s).tile_elems == 4096
        assert_same(engine_results(s, tr), ref, "4096")
    finally:
        hp.hpop_session_destroy(s)
