"""Queries from several host threads on one set and one stream: each call's bounds
and results pass through memory of the handle.  Every result against the oracle."""
import threading

import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_host_queries_from_threads(orc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_05055_amd as cp
    keys = orc.build_set(synth.uniform_keys(200000, 7801, bits=40))
    c = cp.CPMA(keys)
    work = []
    for t, q in enumerate((1, 64, 1000, 1024, 1025, 3000)):  # few queries and more, of different sizes
        lo, hi = synth.range_queries_width(q, 7810 + t, 1 << 33)
        probe = np.concatenate([keys[t::97][:q // 2], lo])[:q]
        work.append((lo, hi, probe, orc.range_map(keys, lo, hi), orc.contains(keys, probe)))
    bad, start = [], threading.Barrier(len(work))

    def client(i):
        lo, hi, probe, (es, en), member = work[i]
        start.wait()
        for _ in range(60):
            s, n = c.range_map(lo, hi)
            if not (np.array_equal(s, es) and np.array_equal(n, en)):
                bad.append(("range_map", len(lo)))
            if not np.array_equal(c.contains(probe), member):
                bad.append(("contains", len(lo)))

    threads = [threading.Thread(target=client, args=(i,)) for i in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not bad, bad[:5]
    c.close()
