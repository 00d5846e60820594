"""Both forms of range_map's end lookups, on either side of the batch size that divides
them: ranges within a leaf, into the next and over several, from below the first key
to past the last, empty and reversed ones; plain, wide, raw and key-value leaves, and
the entry point that allocates nothing.  Exact against the oracle."""
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
    j = np.minimum(i + r.choice([0, 1, 2, 5, 30, 200, 800, 3000], q), len(keys) - 1)
    lo = keys[i] + r.choice(np.array([0, 1, 2**64 - 1], np.uint64), q)
    hi = keys[j] + r.choice(np.array([0, 1, 2, 2**64 - 1], np.uint64), q)
    swap = r.random(q) < 0.03
    lo, hi = np.where(swap, hi, lo), np.where(swap, lo, hi)
    lo[: q // 3: 7] = 0  # below every key, and into every leaf
    hi[q // 2:: 11] = 2**64 - 1
    return lo, hi


@pytest.mark.parametrize("q", [1, 2, 5, 8192, 8193, 40001])
@pytest.mark.parametrize("bits,S,form", [(22, 1024, "plain"), (40, 128, "plain"), (63, 1024, "plain"), (40, 1024, "raw"),
                                         (63, 512, "values"), (22, 2048, "values")])
def test_forms(cp, orc, bits, S, form, q):
    keys = np.unique(synth.uniform_keys(20000, 7980, bits=bits) + np.uint64(9))
    vals = synth.uniform_keys(len(keys), 7981, bits=64) if form == "values" else None
    c = cp.CPMA(keys, leaf_bytes=S, uncompressed=form == "raw", values=vals)
    lo, hi = ranges(keys, q, 7982 + q)
    es, en = orc.range_map(keys, lo, hi)
    s, n = c.range_map(lo, hi)
    assert np.array_equal(n, en) and np.array_equal(s, es)
    if vals is not None:
        K, V = orc.kv_build(keys, vals)
        evs, evn = orc.kv_range_values(K, V, lo, hi)
        s, n = c.range_map_values(lo, hi)
        assert np.array_equal(n, evn) and np.array_equal(s, evs)
    import torch

    def dev(a):
        return torch.from_numpy(np.ascontiguousarray(a, np.uint64).view(np.int64)).cuda()

    s, n = c.range_map_noalloc(dev(lo), dev(hi))
    assert np.array_equal(n.cpu().numpy().view(np.uint64), en)
    assert np.array_equal(s.cpu().numpy().view(np.uint64), es)
    c.close()


def test_statistics_count_the_leaves_read(cp, orc):
    """The scan's bytes: every leaf of a range once, whichever kernel reads it."""
    keys = np.arange(10, 400010, 2, dtype=np.uint64)
    c = cp.CPMA(keys)
    _, used, head = c.export()
    lo, hi = np.array([head[3] + 5], np.uint64), np.array([head[9] + 5], np.uint64)
    c.stats_select(["range_scan"])
    c.range_map(lo, hi)
    got = c.stats()["range_scan"][2]
    c.stats_select([])
    assert got >= int(used[3:10].sum()) and got <= int(used[3:10].sum()) + 64
    c.close()
