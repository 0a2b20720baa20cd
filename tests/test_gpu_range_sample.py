"""Sampled start ranges: chunks at the edge of the sample's size, records in any
order, and starts outside the sampled range (the build is redone), through each
entry point that builds."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu

SPAN = 1 << 31


def trace(n, rng, order="sorted", outlier=None, n_devices=3):
    """n records per resource and kind; `outlier`: the middle record of device 1's kernels starts there."""
    chunks = []
    for r in range(1 + n_devices):
        for k in ((0, 1, 2) if r == 0 else (3, 4)):
            s = tg.T0 + rng.integers(SPAN // 4, 3 * SPAN // 4, size=n)
            s = np.sort(s) if order == "sorted" else s
            e = s + rng.integers(0, SPAN // (2 * n), size=n)
            if outlier is not None and (r, k) == (2, 3):
                s[n // 2] = tg.T0 + outlier
                e[n // 2] = s[n // 2] + 1000
            chunks.append(tg.Chunk(r, k, s, e))
    regions = [(tg.T0, tg.T0 + SPAN), (tg.T0 + SPAN // 3, tg.T0 + SPAN // 2), (tg.T0, tg.T0 + SPAN // 4 + 5)]
    return tg.Trace(1, n_devices, chunks, regions)


def check(tr, tuning=None):
    want = oracle.compute(tr)
    s, keep = new_session(tr, device=True, tuning=tuning)
    try:
        for _ in range(3):
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want)
        assert_same(engine_results(s, tr), want, "without a rebuild")
    finally:
        hp.hpop_session_destroy(s)


@pytest.mark.parametrize("tile", [0, 512, 4096])
@pytest.mark.parametrize("order", ["sorted", "any"])
@pytest.mark.parametrize("n", [1700, 2047, 2048, 2049, 2050, 9000])
def test_chunk_sizes_and_orders(n, order, tile):
    check(trace(n, np.random.default_rng(n), order), {"tile_elems": tile})


# before the sampled range, inside its margin, and after it
@pytest.mark.parametrize("tile", [0, 2048, 8192])
@pytest.mark.parametrize("outlier", [0, SPAN // 4 - SPAN // 512, 3 * SPAN // 4 + SPAN // 512, SPAN - 2000])
def test_starts_outside_the_sample(outlier, tile):
    check(trace(5001, np.random.default_rng(outlier % 1000), "sorted", outlier), {"tile_elems": tile})


def test_outside_and_slots_overflow_and_invalid_together():
    """The redo for the range, then the one for the slots; and an invalid record is still the one named."""
    rng = np.random.default_rng(8)
    tr = trace(6000, rng, "sorted", 0)
    c = tr.chunks[-1]
    c.start[1500:] = tg.T0 + SPAN // 2 + rng.integers(0, 50, size=c.start.size - 1500)
    c.end[:] = np.maximum(c.end, c.start)
    check(tr)
    s, keep = new_session(tr, device=True)
    more = hp.add_chunks(s, [(1, tg.DEV_KERNEL, np.array([tg.T0 + 9]), np.array([tg.T0 + 8]))], device=True)
    try:
        with pytest.raises(hp.HpopError) as ei:
            hp.hpop_metrics_compute_all(s)
        assert ei.value.status == hp.HPOP_E_BAD_INTERVAL and "index 0" in ei.value.message
        assert_same(engine_results(s, tr), oracle.compute(tr), "after the drop")
    finally:
        hp.hpop_session_destroy(s)


def test_new_records_after_a_miss():
    """A session that read every start once goes on with new records, with and without one outside."""
    rng = np.random.default_rng(9)
    s, keep = new_session(trace(5000, rng, "sorted", 0), device=True)
    try:
        hp.hpop_metrics_compute_all(s)
        for outlier in (None, SPAN - 5000):
            tr = trace(5000, rng, "sorted", outlier)
            hp.hpop_clear_events(s)
            keep = hp.add_chunks(s, [(c.resource, c.kind, c.start, c.end) for c in tr.chunks], device=True)
            assert_same(engine_results(s, tr), oracle.compute(tr))
    finally:
        hp.hpop_session_destroy(s)


@pytest.mark.parametrize("outlier", [None, 0])
def test_static_and_batch(outlier):
    rng = np.random.default_rng(10)
    tr = trace(5000, rng, "sorted", outlier)
    want = oracle.compute(tr)
    dev = [(c, torch.from_numpy(c.start).cuda(), torch.from_numpy(c.end).cuda()) for c in tr.chunks]
    torch.cuda.synchronize()
    trees, times = hp.hpop_metrics_compute_static(
        tr.n_hosts, tr.n_devices, [(c.resource, c.kind, a, b) for c, a, b in dev], tr.regions, times=True)
    np.testing.assert_array_equal(np.array([hp.tree_sums(t) for t in trees]), want["sums"])
    np.testing.assert_array_equal(times, want["times"])
    other = trace(3000, rng, "any")
    ss = [new_session(t, device=True) for t in (other, tr, other)]
    try:
        for _ in range(2):
            got = hp.hpop_batch_compute([s for s, _ in ss], hp.HPOP_FORCE_REBUILD)
            for k, t in enumerate((other, tr, other)):
                np.testing.assert_array_equal(np.array([hp.tree_sums(x) for x in got[3 * k:3 * k + 3]]),
                                              oracle.compute(t)["sums"])
    finally:
        for s, _ in ss:
            hp.hpop_session_destroy(s)


@pytest.mark.parametrize("hosts,devices", [(0, 0), (0, 2), (2, 0)])
def test_no_resources_or_records(hosts, devices):
    """Nothing to sample, with the passes apart (timing) and together, alone and in a batch."""
    tr = tg.Trace(hosts, devices, [], [(tg.T0, tg.T0 + 1000)])
    want = oracle.compute(tr)
    full = trace(3000, np.random.default_rng(1))
    s, _ = new_session(tr)
    other, keep = new_session(full, device=True)
    try:
        for on in (0, 1, 0):
            assert hp.lib().hpop_session_enable_timing(s, on) == hp.HPOP_OK
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want)
        got = hp.hpop_batch_compute([s, other], hp.HPOP_FORCE_REBUILD)
        np.testing.assert_array_equal(np.array([hp.tree_sums(got[0])]), want["sums"])
        np.testing.assert_array_equal(np.array([hp.tree_sums(t) for t in got[1:]]), oracle.compute(full)["sums"])
    finally:
        hp.hpop_session_destroy(s)
        hp.hpop_session_destroy(other)
