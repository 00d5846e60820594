"""A few scans of a whole large set: every leaf is summed once for all of them, whether
or not an earlier call had more queries."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


def test_prefix_memory_follows_the_sets_size(orc):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_05055_amd as cp
    for n, taken in ((3_000_000, True), (100_000, False)):
        keys = orc.build_set(synth.uniform_keys(n, 7990, bits=40))
        c = cp.CPMA(keys, leaf_bytes=64)
        L, _ = c.geometry()
        assert (24 * L >= 1 << 22) == taken
        lo, hi = np.arange(25, dtype=np.uint64), np.full(25, 1 << 40, np.uint64)
        c.range_map(lo[:1], hi[:1])
        before = c.bytes_held()
        s, n_keys = c.range_map(lo, hi)
        es, en = orc.range_map(keys, lo, hi)
        assert np.array_equal(n_keys, en) and np.array_equal(s, es)
        assert (c.bytes_held() - before >= 12 * L) == taken
        c.close()
