"""Short ranges, whose two ends mostly lie in one leaf and share its walk: bounds
on, below and above keys, a few keys to a few leaves apart, empty and reversed
ranges among them, ends below the first and past the last key, from one query to
thousands, on narrow and wide leaves, key-value leaves and raw leaves.  Exact
against the oracle."""
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


def ranges(keys, q, seed):
    r = np.random.default_rng(seed)
    i = r.integers(0, len(keys), q)
    d = r.choice([0, 1, 2, 7, 16, 40, 90, 300, 900], q)
    j = np.minimum(i + d, len(keys) - 1)
    lo = keys[i] + r.choice(np.array([0, 1, 2**64 - 1], np.uint64), q)
    hi = keys[j] + r.choice(np.array([0, 1, 2, 2**64 - 1], np.uint64), q)
    swap = r.random(q) < 0.05
    lo, hi = np.where(swap, hi, lo), np.where(swap, lo, hi)
    lo[:1], hi[-1:] = 0, 2**64 - 1
    return lo, hi


@pytest.mark.parametrize("q", [1, 2, 31, 33, 700, 5000])
@pytest.mark.parametrize("bits,S", [(18, 64), (40, 1024), (40, 4096), (63, 1024), (63, 256)])
def test_keys(cp, orc, bits, S, q):
    print(f"[range pairs] bits={bits} S={S} q={q}", flush=True)
    keys = orc.build_set(synth.uniform_keys(30000, 71, bits=bits) + np.uint64(5))
    lo, hi = ranges(keys, q, 72 + q)
    want = orc.range_map(keys, lo, hi)
    for raw in (0, 1):
        cfg = cp.default_config()
        cfg.leaf_bytes, cfg.uncompressed = S, raw
        c = cp.CPMA(keys, config=cfg)
        s, n = c.range_map(lo, hi)
        assert np.array_equal(n, want[1]) and np.array_equal(s, want[0]), raw
        c.close()


@pytest.mark.parametrize("q", [2, 33, 5000])
@pytest.mark.parametrize("bits,S", [(40, 1024), (63, 256)])
def test_values(cp, orc, bits, S, q):
    print(f"[range pairs] values bits={bits} S={S} q={q}", flush=True)
    keys = np.unique(synth.uniform_keys(30000, 73, bits=bits) + np.uint64(5))
    vals = synth.uniform_keys(len(keys), 74, bits=64)
    c = cp.CPMA(keys, leaf_bytes=S, values=vals)
    K, V = orc.kv_build(keys, vals)
    lo, hi = ranges(keys, q, 75 + q)
    s, n = c.range_map(lo, hi)
    es, en = orc.range_map(K, lo, hi)
    assert np.array_equal(n, en) and np.array_equal(s, es)
    vs, vn = c.range_map_values(lo, hi)
    evs, evn = orc.kv_range_values(K, V, lo, hi)
    assert np.array_equal(vn, evn) and np.array_equal(vs, evs)
