"""range_map around the switch to per-leaf prefix sums: batches that visit fewer
and more interior leaves than the set has, at few and many queries (the
prefix pass finishes up to 64 queries itself), around its steps of 32 leaves, on
key spans below 2^28, below 2^32 and above per leaf, for every leaf format.
Exact against the oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

M64 = (1 << 64) - 1


@pytest.fixture(scope="module")
def cp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_05055_amd as p
    p.lib()
    return p


def queries(keys, q, share, seed, bits):
    """q ranges over about `share` of the set each, empty and full ones among them."""
    lo = synth.uniform_keys(q, seed, bits=bits)
    hi = lo + np.uint64(int(share * ((1 << bits) - 1)))
    hi = np.where(hi < lo, np.uint64(M64), hi)
    lo[0], hi[0] = 0, M64
    if q > 2:
        lo[1], hi[1] = keys[len(keys) // 2], keys[len(keys) // 2]
    return lo, hi


@pytest.mark.parametrize("q", [2, 3, 64, 65, 3000])
@pytest.mark.parametrize("S,n,bits", [(64, 3000, 40), (64, 1, 40), (128, 9000, 28), (1024, 60000, 40), (1024, 40000, 34),
                                      (1024, 30000, 63), (4096, 200000, 40)])
def test_prefix_and_direct(cp, orc, S, n, bits, q):
    keys = orc.build_set(synth.uniform_keys(n, 5100 + n, bits=bits))
    sets = {"plain": cp.CPMA(keys, leaf_bytes=S), "raw": cp.CPMA(keys, leaf_bytes=S, uncompressed=True)}
    for share in (0.0005, 0.6):
        lo, hi = queries(keys, q, share, 5200 + q, bits)
        es, en = orc.range_map(keys, lo, hi)
        for name, c in sets.items():
            s, m = c.range_map(lo, hi)
            assert np.array_equal(m, en) and np.array_equal(s, es), (name, share)
    for c in sets.values():
        c.close()


@pytest.mark.parametrize("S,n", [(128, 5000), (1024, 30000)])
@pytest.mark.parametrize("q", [5, 2000])
def test_prefix_values(cp, orc, S, n, q):
    keys = synth.uniform_keys(n, 5300 + n, bits=40)
    vals = synth.uniform_keys(n, 5301 + n, bits=64)
    K, V = orc.kv_build(keys, vals)
    c = cp.CPMA(keys, leaf_bytes=S, values=vals)
    for share in (0.0005, 0.6):
        lo, hi = queries(K, q, share, 5400 + q, 40)
        s, m = c.range_map(lo, hi)
        es, en = orc.range_map(K, lo, hi)
        assert np.array_equal(m, en) and np.array_equal(s, es)
        vs, vm = c.range_map_values(lo, hi)
        evs, evn = orc.kv_range_values(K, V, lo, hi)
        assert np.array_equal(vm, evn) and np.array_equal(vs, evs)
    c.close()


def test_prefix_follows_growth(cp, orc):
    """The prefixes belong to one call: updates in between, with growth, change every answer."""
    keys = orc.build_set(synth.uniform_keys(20000, 5500, bits=40))
    c = cp.CPMA(keys, leaf_bytes=256)
    for step in range(4):
        lo, hi = queries(keys, 1500, 0.5, 5600 + step, 40)
        s, m = c.range_map(lo, hi)
        es, en = orc.range_map(keys, lo, hi)
        assert np.array_equal(m, en) and np.array_equal(s, es)
        batch = synth.uniform_keys(15000, 5700 + step, bits=40)
        c.insert_batch(batch)
        keys, _ = orc.insert(keys, batch)
    c.close()
