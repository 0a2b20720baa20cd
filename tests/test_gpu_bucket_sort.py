"""The orders a bucket's records can take through the sorts of the merge: one
count of sub-bins, a second count where starts lie in a few places, the
insertion sort's largest sub-bin and the radix sort behind it, in the wave
path (8 B records) and the block path (more records, wide buckets)."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu


def trace(starts, rng, mean):
    """The same starts on a host and two devices, in another order on each, with ends of a few lengths."""
    span = int(starts.max()) + 4 * mean + 4
    chunks = []
    for r in range(3):
        s = tg.T0 + rng.permutation(starts)
        e = s + rng.integers(0, 4 * mean, size=s.size)
        k = rng.integers(0, 3 if r == 0 else 2, size=s.size) + (0 if r == 0 else 3)
        chunks += [tg.Chunk(r, int(q), s[k == q], e[k == q]) for q in np.unique(k)]
    regions = [(tg.T0, tg.T0 + span), (tg.T0 + span // 3, tg.T0 + span // 2 + 1), (tg.T0 + 1, tg.T0 + 2)]
    return tg.Trace(1, 2, chunks, regions)


def check(tr, tuning):
    want = oracle.compute(tr)
    s, keep = new_session(tr, device=True, tuning=tuning)
    try:
        for _ in range(2):
            assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want)
    finally:
        hp.hpop_session_destroy(s)


def clusters(rng, n, span, places, width):
    at = rng.integers(0, max(1, span - width), size=places)
    return at[rng.integers(0, places, size=n)] + rng.integers(0, width, size=n)


# one bucket per resource (the bucket target is the largest), so the records of a bucket are those given
@pytest.mark.parametrize("wide", [False, True], ids=["narrow", "wide"])
@pytest.mark.parametrize("n", [2, 9, 65, 449, 512, 513, 1500, 2047])
@pytest.mark.parametrize("shape", ["even", "two places", "ten places", "equal pairs", "equal crowd", "one far"])
def test_orders(n, shape, wide):
    rng = np.random.default_rng(n * 7 + len(shape) + wide)
    span = (1 << 40) if wide else (1 << 29)
    if shape == "even":
        st = rng.integers(0, span, size=n)
    elif shape == "two places":
        st = clusters(rng, n, span, 2, 50_000)
    elif shape == "ten places":
        st = clusters(rng, n, span, 10, 1_000)
    elif shape == "equal pairs":
        st = np.repeat(rng.integers(0, span, size=n // 2 + 1), 2)[:n]
    elif shape == "equal crowd":  # one sub-bin with more equal starts than any insertion sort takes
        st = np.where(rng.random(n) < 0.5, span // 3, rng.integers(0, span, size=n))
    else:  # every start but one within a microsecond
        st = rng.integers(0, 1000, size=n)
        st[-1] = span
    st = np.sort(st) - st.min()
    check(trace(st, rng, max(2, int(span // (4 * n)))), {"bucket_target": 4096, "scatter_slots": 2048, "tile_elems": 2048})


def test_many_wide_buckets():
    """Every bucket through the block path's lists: more than one per workgroup."""
    rng = np.random.default_rng(5)
    n = 30_000
    st = np.sort(rng.integers(0, n << 28, size=n))
    check(trace(st, rng, 1 << 28), {"bucket_target": 16})


@pytest.mark.parametrize("extra", [0, 1])
def test_tile_size_changes_with_the_records(extra):
    """The most records of a build with the smallest tiles, and one more (three resources, the last ones of a tile each)."""
    n = (128 << 10) // 3
    rng = np.random.default_rng(extra)
    tr = trace(np.sort(rng.integers(0, n * 60_000, size=n)), rng, 60_000)
    more = (128 << 10) - 3 * n + extra
    tr.chunks += [tg.Chunk(1, tg.DEV_KERNEL, tg.T0 + np.arange(more), tg.T0 + np.arange(more) + 5)]
    check(tr, {})


@pytest.mark.parametrize("devices,buckets", [(1, 127), (1, 129), (2, 341), (2, 342), (1, 1025), (0, 66_000), (300, 64)])
def test_bucket_counts(devices, buckets):
    """Edges of the bucket passes: workgroup per segment or wave, one tile of 1024 buckets and more, over 64 tiles."""
    rng = np.random.default_rng(devices + buckets)
    n = 16 * buckets
    chunks = []
    for r in range(1 + devices):
        s = tg.T0 + np.sort(rng.integers(0, n * 1000, size=n))
        chunks.append(tg.Chunk(r, 2 if r == 0 else 3, s, s + rng.integers(0, 1500, size=n)))
    regions = [(tg.T0, tg.T0 + n * 1000), (tg.T0 + n * 300, tg.T0 + n * 700 + 1)]
    check(tg.Trace(1, devices, chunks, regions), {"bucket_target": 16})
