"""Records in bursts of close but different starts, which crowd even in the
second count's parts: sorted by the wave that has the bucket."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results, new_session

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [60, 66, 130, 256, 300, 500, 512, 700, 20_000])
@pytest.mark.parametrize("burst,width", [(24, 1000), (40, 50), (33, 2), (200, 100_000)])
def test_bursts(burst, width, n):
    """Alone in one bucket (n of a wave's sizes, at and past its largest), and over many buckets; with records
    that reach past the bucket, in one kernel (n <= 4096) and by passes."""
    rng = np.random.default_rng(burst + n)
    mean = 45_000
    chunks = []
    for r in range(6):
        s = np.repeat(rng.integers(0, n * mean, size=n // burst + 1), burst)[:n] + rng.integers(0, width, size=n)
        s = tg.T0 + rng.permutation(s)
        e = s + rng.integers(0, 2 * mean, size=n) * np.where(rng.random(n) < 0.02, 200, 1)
        k = rng.integers(0, 3 if r < 2 else 2, size=n) + (0 if r < 2 else 3)
        chunks += [tg.Chunk(r, int(q), s[k == q], e[k == q]) for q in np.unique(k)]
    end = tg.T0 + n * mean
    tr = tg.Trace(2, 4, chunks, [(tg.T0, end + 400 * mean), (tg.T0 + n * mean // 3, tg.T0 + n * mean // 2)])
    print("case: n=%d burst=%d width=%d" % (n, burst, width), flush=True)
    want = oracle.compute(tr)
    for timed in (False, True):  # timed builds run as separate passes
        s, keep = new_session(tr, device=True, tuning={"bucket_target": 512 if n <= 512 else 0})
        try:
            hp.hpop_session_enable_timing(s, timed)
            for _ in range(2):
                assert_same(engine_results(s, tr, hp.HPOP_FORCE_REBUILD), want, "timed %s" % timed)
        finally:
            hp.hpop_session_destroy(s)
