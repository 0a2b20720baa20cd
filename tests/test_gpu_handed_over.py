"""Buckets that the wave path hands over, in builds that run as separate passes
(a resource of more than 4096 records, so that no workgroup takes a whole
resource): crowded sub-bins, many equal starts, wide buckets and buckets of
more than 512 records side by side in one workgroup's list."""
import time

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu


def resource(r, starts, rng, mean):
    host = r[1]
    e = starts + rng.integers(0, 4 * mean, size=starts.size)
    k = rng.integers(0, 3 if host else 2, size=starts.size) + (0 if host else 3)
    return [tg.Chunk(r[0], int(q), starts[k == q], e[k == q]) for q in np.unique(k)]


def check(tr, tuning=None):
    print("case: records=%d tuning=%s" % (tr.n_events, tuning), flush=True)
    want = oracle.compute(tr)
    s, keep = new_session(tr, device=True, tuning=tuning)
    try:
        for _ in range(3):
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want)
    finally:
        hp.hpop_session_destroy(s)


def regions(t1):
    return [(tg.T0, t1), (tg.T0 + (t1 - tg.T0) // 3, tg.T0 + (t1 - tg.T0) // 2 + 1), (tg.T0 + 1, tg.T0 + 2)]


@pytest.mark.parametrize("tick_ms", [1, 2])
@pytest.mark.parametrize("mean_us", [30, 45, 60])
def test_coarse_clock(mean_us, tick_ms):
    """Starts on a clock of 1 or 2 ms: every bucket has crowded sub-bins, some or all of more equal starts
    than the second count and the insertion sort take."""
    rng = np.random.default_rng(mean_us * 10 + tick_ms)
    mean, tick, n = mean_us * 1000, tick_ms * 1_000_000, 20_011
    chunks = []
    for r in range(6):
        s = np.sort(rng.integers(0, n * mean, size=n)) // tick * tick + tg.T0
        chunks += resource((r, r < 2), s, rng, mean)
    check(tg.Trace(2, 4, chunks, regions(tg.T0 + n * mean)))


@pytest.mark.parametrize("equal", [False, True], ids=["ns", "2 ms"])
def test_wide_hosts_beside_phased_devices(equal):
    """Hosts with few records over minutes (16 B records), devices active in phases of 20 ms every 330 ms
    (crowded sub-bins; with equal starts the second count fails too): both in every workgroup's list."""
    rng = np.random.default_rng(3 + equal)
    span = 100_000_000_000
    chunks = []
    for r in range(16):
        if r < 8:
            s = np.sort(rng.integers(0, span, size=5003))  # buckets of 6 s
            mean = 10_000_000
        else:
            s = rng.integers(0, span // 330_000_000, size=50_021) * 330_000_000 + rng.integers(0, 20_000_000, size=50_021)
            s = np.sort(s // 2_000_000 * 2_000_000 if equal else s)
            mean = 50_000
        chunks += resource((r, r < 8), tg.T0 + s, rng, mean)
    check(tg.Trace(8, 8, chunks, regions(tg.T0 + span)))


def starts_of(shape, n, span, rng):
    if shape == "even":
        st = rng.integers(0, span, size=n)
    elif shape == "two places":
        st = rng.integers(0, span - 50_000, size=2)[rng.integers(0, 2, size=n)] + rng.integers(0, 50_000, size=n)
    elif shape == "ten places":
        st = rng.integers(0, span - 1_000, size=10)[rng.integers(0, 10, size=n)] + rng.integers(0, 1_000, size=n)
    elif shape == "equal pairs":
        st = np.repeat(rng.integers(0, span, size=n // 2 + 1), 2)[:n]
    elif shape == "equal crowd":  # more equal starts than any insertion sort takes
        st = np.where(rng.random(n) < 0.5, span // 3, rng.integers(0, span, size=n))
    else:  # every start but one within a microsecond
        st = rng.integers(0, 1000, size=n)
        st[-1] = span
    return np.sort(st) - st.min()


# one bucket per resource but the last, which has more than 4096 records
@pytest.mark.parametrize("cap", [2048, 4096])
@pytest.mark.parametrize("wide", [False, True], ids=["narrow", "wide"])
@pytest.mark.parametrize("n", [2, 9, 65, 449, 512, 513, 1500, 2047])
def test_orders_by_passes(n, wide, cap):
    """Every shape and form of a bucket's starts in one build."""
    rng = np.random.default_rng(n * 7 + wide + cap)
    shapes = ["even", "two places", "ten places", "equal pairs", "equal crowd", "one far"]
    chunks, devices = [], 0
    for i, shape in enumerate(shapes * 3):
        # with wide buckets among them, every other resource has narrow ones
        span = (1 << 40) if wide and i % 2 else (1 << 29)
        st = starts_of(shape, n, span, rng)
        chunks += resource((i, i < 6), tg.T0 + rng.permutation(st), rng, max(2, int(span // (4 * n))))
        devices += i >= 6
    many = np.sort(rng.integers(0, 1 << 29, size=4500))
    chunks += resource((len(shapes) * 3, False), tg.T0 + many, rng, 50_000)
    check(tg.Trace(6, devices + 1, chunks, regions(tg.T0 + (1 << 40 if wide else 1 << 29) + 100)),
          {"bucket_target": 2047, "bucket_cap": cap, "scatter_slots": cap, "tile_elems": 2048})


@pytest.mark.parametrize("passes", [True, False], ids=["passes", "one kernel"])
@pytest.mark.parametrize("wide", [False, True], ids=["narrow", "wide"])
@pytest.mark.parametrize("c", [15, 16, 17, 32, 33, 34, 200, 505, 1200])
def test_crowds_of_equal_starts(c, wide, passes):
    """c records of one start, of every kind and any length, alone in their sub-bin and with one start beside
    them before or after: equal starts need no sort, a crowd with another start does."""
    rng = np.random.default_rng(c + wide)
    span = (1 << 40) if wide else (1 << 29)
    chunks = []
    for i in range(4):
        s = np.full(c, span // 2, np.int64)
        near = [np.zeros(0, np.int64), np.array([span // 2 - 1]), np.array([span // 2 + 1]),
                np.array([span // 2 - 1, span // 2 + 3])][i]
        s = np.concatenate([s, near, rng.integers(0, span, size=7), [0, span - 1]])
        chunks += resource((i, i < 2), tg.T0 + rng.permutation(s), rng, int(span // 4 // (1 + i)))
    n_devices = 2
    if passes:
        chunks += resource((4, False), tg.T0 + np.sort(rng.integers(0, 1 << 29, size=4500)), rng, 50_000)
        n_devices = 3
    check(tg.Trace(2, n_devices, chunks, regions(tg.T0 + 2 * span)),
          {"bucket_target": 2047, "scatter_slots": 2048, "tile_elems": 2048})


def test_equal_starts_cost_no_sort():
    """A coarse clock's records take about as long as the same ones in ns (1.1 times with starts of 1 ms, where
    a sort of every crowd took 5.6 times as long)."""
    rng = np.random.default_rng(11)
    n, mean, R = 60_000, 45_000, 64
    took = []
    for tick in (1, 1_000_000):
        chunks = []
        for r in range(R):
            s = tg.T0 + np.sort(rng.integers(0, n * mean, size=n)) // tick * tick
            chunks.append(tg.Chunk(r, tg.DEV_KERNEL, s, s + rng.integers(0, 2 * mean, size=n)))
        s, keep = new_session(tg.Trace(0, R, chunks, [(tg.T0, tg.T0 + n * mean)]), device=True)
        try:
            v = []
            for _ in range(25):
                t = time.perf_counter()
                hp.hpop_metrics_compute_all(s, hp.HPOP_FORCE_REBUILD)
                v.append(time.perf_counter() - t)
            took.append(sorted(v)[12])
        finally:
            hp.hpop_session_destroy(s)
    print("ns %.1f us, 1 ms %.1f us" % (1e6 * took[0], 1e6 * took[1]), flush=True)
    assert took[1] < 2 * took[0]
