"""Builds whose segments are all small (one workgroup per segment): sizes at
the edges of a round of records, a bucket, a kernel variant and the path
itself, and the cases that leave its common branch."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu


def trace(n, rng, n_devices=2, span_per=70_000, chunks_per=1):
    """One host and devices with n records each, delivered in time order."""
    span = max(4, n * span_per)
    chunks = []
    for r in range(1 + n_devices):
        s = np.sort(tg.T0 + rng.integers(0, span, size=n))
        e = s + rng.integers(0, 2 * span_per, size=n)
        k = rng.integers(0, 3 if r == 0 else 2, size=n) + (0 if r == 0 else 3)
        for kind in np.unique(k):
            for part in np.array_split(np.flatnonzero(k == kind), chunks_per):
                if part.size:
                    chunks.append(tg.Chunk(r, int(kind), s[part], e[part]))
    regions = [(tg.T0, tg.T0 + span), (tg.T0 + span // 3, tg.T0 + span // 2 + 1), (tg.T0 - 5, tg.T0 + 1)]
    return tg.Trace(1, n_devices, chunks, regions)


def check(tr, tuning=None):
    want = oracle.compute(tr)
    s, keep = new_session(tr, device=True, tuning=tuning)
    try:
        for _ in range(3):  # launched one by one, then captured, then replayed
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want)
        return hp.hpop_session_get_info(s)
    finally:
        hp.hpop_session_destroy(s)


@pytest.mark.parametrize("n", [1, 64, 351, 353, 511, 513, 1025, 4095, 4096, 4097])
def test_sizes(n):
    check(trace(n, np.random.default_rng(n)))


@pytest.mark.parametrize("per", [1, 40, 42, 63, 64])
def test_many_chunks_per_segment(per):
    """Up to 128 chunks per segment take the path; 3 x 63 of the host do not."""
    check(trace(3000, np.random.default_rng(per), chunks_per=per))


@pytest.mark.parametrize("target", [16, 64, 2048])
def test_bucket_targets(target):
    """A few buckets, as many as the path takes (and more), and large ones for the block path."""
    check(trace(1020, np.random.default_rng(target)), tuning={"bucket_target": target})


def test_resources_without_records_and_unequal_ones():
    rng = np.random.default_rng(3)
    tr = trace(900, rng, n_devices=5)
    tr.chunks = [c for c in tr.chunks if c.resource not in (2, 4)]
    tr.chunks.append(tg.Chunk(4, tg.DEV_KERNEL, np.array([tg.T0 + 7]), np.array([tg.T0 + 7])))  # covers nothing
    check(tr)


def test_wide_buckets_far_ends_and_crowded_starts():
    rng = np.random.default_rng(4)
    wide = trace(700, rng, n_devices=1, span_per=20_000_000)  # buckets wider than 2^30 ns: the 16 B form
    assert check(wide).n_wide_records > 0
    far = trace(4000, rng)
    c = far.chunks[-1]
    c.end = c.end.copy()
    c.end[::97] += 1 << 34  # clamped in the 8 B form
    check(far)
    crowd = trace(1500, rng)
    c = crowd.chunks[-1]
    c.start = c.start.copy()
    c.start[: c.start.size // 2] = tg.T0 + 12345 + np.arange(c.start.size // 2) % 50
    c.end = np.maximum(c.end, c.start)
    check(crowd)


def test_slot_overflow_redoes_the_build():
    rng = np.random.default_rng(6)
    tr = trace(4000, rng)
    c = tr.chunks[-1]
    c.start = c.start.copy()
    c.start[100:] = tg.T0 + 1_000_000 + rng.integers(0, 60, size=c.start.size - 100)
    c.end = np.maximum(c.end, c.start)
    check(tr)


def test_invalid_record_is_named_and_dropped():
    rng = np.random.default_rng(7)
    tr = trace(3000, rng)
    bad = tg.Chunk(1, tg.DEV_KERNEL, np.array([tg.T0 + 5, tg.T0 + 9]), np.array([tg.T0 + 6, tg.T0 + 8]))
    s, keep = new_session(tr, device=True)
    more = hp.add_chunks(s, [(bad.resource, bad.kind, bad.start, bad.end)], device=True)
    try:
        with pytest.raises(hp.HpopError) as ei:
            hp.hpop_metrics_compute_all(s)
        assert ei.value.status == hp.HPOP_E_BAD_INTERVAL and "index 1" in ei.value.message
        assert_same(engine_results(s, tr), oracle.compute(tr), "after the drop")
    finally:
        hp.hpop_session_destroy(s)


@pytest.mark.parametrize("devices", [511, 512])
def test_most_segments_of_the_path_and_one_more(devices):
    check(trace(70, np.random.default_rng(devices), n_devices=devices))
