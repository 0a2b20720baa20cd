"""Sets of records with and without a start outside its sampled range, in one
session and in a batch that goes on: every answer is the oracle's."""
import time

import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu

SPAN = 1 << 31


def trace(rng, outlier, n=5000):
    """Two devices, evenly spread starts; the middle record of device 0 starts at `outlier`, if given."""
    chunks = []
    for r in range(2):
        s = np.sort(tg.T0 + rng.integers(SPAN // 4, 3 * SPAN // 4, size=n))
        e = s + rng.integers(0, SPAN // n, size=n)
        if r == 0 and outlier is not None:
            s[n // 2] = tg.T0 + outlier
            e[n // 2] = s[n // 2] + 1000
        chunks.append(tg.Chunk(r, tg.DEV_KERNEL, s, e))
    return tg.Trace(0, 2, chunks, [(tg.T0, tg.T0 + SPAN), (tg.T0, tg.T0 + SPAN // 4)])


def add(s, tr):
    return hp.add_chunks(s, [(c.resource, c.kind, c.start, c.end) for c in tr.chunks], device=True)


@pytest.mark.parametrize("row", [[0, None, None], [0, SPAN - 9, 5, 0, 0, None, None, None, None, 3]], ids=["one", "row"])
def test_session_and_batch_go_on(row):
    rng = np.random.default_rng(len(row))
    keep = [new_session(trace(rng, None), device=True) for _ in range(2)]
    ss = [s for s, _ in keep]
    try:
        for outlier in row:
            trs = [trace(rng, outlier), trace(rng, None)]
            for s, tr in zip(ss, trs):
                hp.hpop_clear_events(s)
                keep.append(add(s, tr))
            wants = [oracle.compute(tr) for tr in trs]
            for flags in (0, hp.HPOP_FORCE_REBUILD):
                got = hp.hpop_batch_compute(ss, flags)
                for k in range(2):
                    np.testing.assert_array_equal(np.array([hp.tree_sums(t) for t in got[2 * k:2 * k + 2]]), wants[k]["sums"])
                for s, tr, want in zip(ss, trs, wants):
                    assert_same(engine_results(s, tr, flags), want, "outlier %s" % outlier)
        # more records on top of those that missed
        extra = trace(rng, None, 4000)
        keep.append(add(ss[0], extra))
        both = tg.Trace(0, 2, trs[0].chunks + extra.chunks, extra.regions)
        assert_same(engine_results(ss[0], both), oracle.compute(both))
    finally:
        for s in ss:
            hp.hpop_session_destroy(s)


def test_static_calls_build_once():
    """Calls that share nothing don't pay for a start apart from the others: with one they take
    as long as without (1.0-1.1 times; building twice takes 1.8 times as long)."""
    rng = np.random.default_rng(4)
    n, R, span = 60_000, 16, 60_000 * 60_000
    calls, wants = [], []
    for outlier in (False, True):
        chunks = []
        for r in range(R):
            s = tg.T0 + span // 8 + np.sort(rng.integers(0, span, size=n))
            if outlier and r == 0:
                s[n // 2] = tg.T0 + span // 16
            chunks.append(tg.Chunk(r, tg.DEV_KERNEL, s, s + rng.integers(0, 60_000, size=n)))
        tr = tg.Trace(0, R, chunks, [(tg.T0, tg.T0 + 2 * span)])
        dev = [(c.resource, c.kind, torch.from_numpy(c.start).cuda(), torch.from_numpy(c.end).cuda()) for c in chunks]
        calls.append((dev, tr.regions))
        wants.append(oracle.compute(tr)["sums"])
    torch.cuda.synchronize()
    took = ([], [])
    for _ in range(41):
        for k, (dev, regs) in enumerate(calls):
            t = time.perf_counter()
            trees = hp.hpop_metrics_compute_static(0, R, dev, regs)
            took[k].append(time.perf_counter() - t)
            np.testing.assert_array_equal(np.array([hp.tree_sums(x) for x in trees]), wants[k])
    plain, odd = (sorted(v)[20] for v in took)
    print("static: %.1f us, with a start apart %.1f us" % (1e6 * plain, 1e6 * odd), flush=True)
    assert odd < 1.5 * plain
