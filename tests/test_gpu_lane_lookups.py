"""Lookups with a lane each, in leaves of at most 256 bytes, on either side of the batch
sizes from which they are taken: membership and ranges on narrow and wide leaves, of
keys of plain and key-value sets and through fused requests.  Against the oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_05055_amd as p
    p.lib()
    return p


@pytest.mark.parametrize("S,bits,values", [(64, 22, False), (64, 63, False), (128, 40, False), (256, 40, False),
                                           (256, 63, True), (128, 30, True)])
def test_lookups(cp, orc, S, bits, values):
    keys = np.unique(synth.uniform_keys(50_000, 8200, bits=bits) + np.uint64(3))
    c = cp.CPMA(keys, leaf_bytes=S, values=keys if values else None)
    r = np.random.default_rng(8201)
    for q in (384 * S - 1, 384 * S, 6 * S * S - 1, 6 * S * S):
        i = r.integers(0, len(keys), q)
        lo = keys[i] + r.choice(np.array([0, 1, 2**64 - 1], np.uint64), q)
        hi = keys[np.minimum(i + r.choice([0, 1, 2, 10, 90, 600], q), len(keys) - 1)] + np.uint64(1)
        lo[:q // 4:97], hi[q // 2::101] = 0, 2**64 - 1
        lo[5], hi[6] = 2**64 - 1, 0
        es, en = orc.range_map(keys, lo, hi)
        s, n = c.range_map(lo, hi)
        assert np.array_equal(n, en) and np.array_equal(s, es), q
        assert np.array_equal(c.contains(lo), orc.contains(keys, lo)), q
    c.close()


def test_fused_requests(cp, orc):
    """Fewer keys than leaves, so that membership is looked up per key."""
    keys = np.unique(synth.uniform_keys(1_500_000, 8202, bits=40))
    c = cp.CPMA(keys, leaf_bytes=64)
    batches = [synth.uniform_keys(50_000, 8203, bits=40), keys[::30].copy()]
    assert sum(map(len, batches)) < c.geometry()[0]
    expect, added = orc.insert(keys, batches[0])
    expect, removed = orc.delete(expect, batches[1])
    got = c.apply_updates([(cp.REQ_INSERT, batches[0]), (cp.REQ_DELETE, batches[1])])
    assert list(got) == [added, removed] and c.size() == len(expect)
    c.close()
