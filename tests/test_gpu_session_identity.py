"""A batch keeps its plan while its sessions are unchanged: a session made where a
destroyed one was, with as many calls made, is another session."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is loaded before the library's)

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import new_session

pytestmark = pytest.mark.gpu


def test_batch_with_a_new_session_in_a_destroyed_ones_place():
    rng = np.random.default_rng(6)

    def trace():
        s = tg.T0 + np.sort(rng.integers(0, 1 << 28, size=3000))
        return tg.Trace(0, 1, [tg.Chunk(0, tg.DEV_KERNEL, s, s + rng.integers(0, 1 << 17, size=3000))],
                        [(tg.T0, tg.T0 + (1 << 28)), (tg.T0 + 5, tg.T0 + (1 << 27))])

    first = trace()
    lead, _ = new_session(first)
    try:
        for _ in range(6):
            tr = trace()
            other, _ = new_session(tr)
            got = hp.hpop_batch_compute([lead, other], 0)
            for k, t in enumerate((first, tr)):
                np.testing.assert_array_equal(np.array([hp.tree_sums(x) for x in got[2 * k:2 * k + 2]]),
                                              oracle.compute(t)["sums"])
            hp.hpop_session_destroy(other)
    finally:
        hp.hpop_session_destroy(lead)
