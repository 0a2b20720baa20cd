"""Chunks whose records come in pieces, each in the order of time but not one
after another (several threads' or streams' records put together, a ring that
wrapped): the sample sees the pieces between a chunk's ends too, so that the
build needs no exact offsets; and a stretch of records that it cannot see."""
import numpy as np
import pytest

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu

MEAN = 1000  # ns from one start to the next


def stages(tr):
    s, keep = new_session(tr, device=True)
    try:
        hp.hpop_session_enable_timing(s, True)
        want = oracle.compute(tr)
        assert_same(engine_results(s, tr), want)
        names = [n for n, _ in hp.hpop_session_stage_times(s)]
        assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want, "again")
        return names
    finally:
        hp.hpop_session_destroy(s)


@pytest.mark.parametrize("n", [1535, 1536, 1537, 1600, 9001, 60_000, 200_003])
@pytest.mark.parametrize("pieces", [[1, 0], [0, 2, 1], [2, 0, 3, 1], [4, 3, 2, 1, 0]],
                         ids=["wrapped", "middle last", "four", "backwards"])
def test_pieces_in_another_order(pieces, n):
    rng = np.random.default_rng(n + len(pieces))
    chunks = []
    for r in range(3):
        s = tg.T0 + np.sort(rng.integers(0, n * MEAN, size=n))
        e = s + rng.integers(0, 2 * MEAN, size=n)
        cut = np.linspace(0, n, len(pieces) + 1).astype(int)
        at = np.concatenate([np.arange(cut[p], cut[p + 1]) for p in pieces])
        chunks.append(tg.Chunk(r, tg.HOST_USEFUL if r == 0 else tg.DEV_KERNEL, s[at], e[at]))
    end = tg.T0 + n * MEAN
    names = stages(tg.Trace(1, 2, chunks, [(tg.T0, end + 5), (tg.T0 + n * MEAN // 3, end - n * MEAN // 5)]))
    assert "hist" not in names


@pytest.mark.parametrize("past", [False, True], ids=["before", "past"])
def test_tiles_outside_from_end_to_end(past):
    """More records than a tile's between two of the sampled ones start elsewhere: the build with exact offsets."""
    n = 600_000
    rng = np.random.default_rng(6)
    s = tg.T0 + (1 << 40) + np.sort(rng.integers(0, n * MEAN, size=n))
    hop = (n - 1032) // 64
    at = 512 + hop // 2 + 30 * hop + 8  # past the run of 8 that is sampled there
    s[at:at + hop - 8] += (1 << 39) if past else -(1 << 39)
    e = s + rng.integers(0, 2 * MEAN, size=n)
    tr = tg.Trace(0, 1, [tg.Chunk(0, tg.DEV_KERNEL, s, e)],
                  [(int(s.min()), int(e.max())), (int(s[at]) + 9, int(s[at]) + 12345), (int(s[0]), int(s[n // 2]))])
    assert "hist" in stages(tr)
