"""Records added from device memory: any number of chunks per call, any size
and word alignment, one allocation or several."""
import numpy as np
import pytest
import torch

import oracle
import paper_2603_26576_amd as hp
import tracegen as tg
from engine_util import assert_same, engine_results

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [[1], [4095, 4096, 4097, 8192, 12291], [7] * 80, [64] * 81,
                                   [1, 0, 4096] * 55], ids=["one", "piece edges", "80", "81", "165"])
@pytest.mark.parametrize("offset", [0, 1], ids=["aligned", "odd word"])
@pytest.mark.parametrize("apart", [False, True], ids=["one allocation", "own allocations"])
def test_device_chunks_match_the_oracle(sizes, offset, apart):
    rng = np.random.default_rng(len(sizes) * 2 + offset)
    n_hosts, n_devices = 2, 3
    kinds = [(r, k) for r in range(n_hosts) for k in (0, 1, 2)] + [(r + n_hosts, k) for r in range(n_devices) for k in (3, 4)]
    chunks = []
    for i, n in enumerate(sizes):
        r, k = kinds[i % len(kinds)]
        s = tg.T0 + rng.integers(0, 10_000_000, size=n)
        chunks.append(tg.Chunk(r, k, s, s + rng.integers(0, 3000, size=n)))
    tr = tg.Trace(n_hosts, n_devices, chunks, [(tg.T0, tg.T0 + 10_000_000), (tg.T0 + 1234, tg.T0 + 7_654_321)])
    dev = []
    if apart:
        for c in chunks:
            buf = [torch.from_numpy(np.concatenate([np.zeros(offset, np.int64), x])).cuda() for x in (c.start, c.end)]
            dev.append((c.resource, c.kind, buf[0][offset:], buf[1][offset:]))
    else:
        flat = [torch.from_numpy(np.concatenate([np.zeros(offset, np.int64)] + [getattr(c, f) for c in chunks])).cuda()
                for f in ("start", "end")]
        at = offset
        for c in chunks:
            n = c.start.size
            dev.append((c.resource, c.kind, flat[0][at:at + n], flat[1][at:at + n]))
            at += n
    torch.cuda.synchronize()
    s = hp.hpop_session_create(n_hosts, n_devices)
    try:
        hp.hpop_add_events_multi(s, dev, hp.HPOP_MEM_DEVICE)
        for a, b in tr.regions:
            hp.hpop_region_define(s, a, b)
        assert_same(engine_results(s, tr), oracle.compute(tr))
    finally:
        hp.hpop_session_destroy(s)
