"""Point lookups (contains, get) and the partial end leaves of range_map at the
edges of the row decoder: leaf heads and their neighbours, the first and last
keys, the reserved key, codes of 1 to 10 bytes across 16- and 256-byte
boundaries, 32- and 64-bit spans, and batches around the number of lookups a
wave takes.  Exact against the oracle."""
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


def key_set(kind, n):
    if kind == "dense":
        k = np.arange(5, 5 + n, dtype=np.uint64)  # one-byte codes
    elif kind == "mixed":  # deltas of every code length, 1 to 9 bytes
        bits = 1 + (np.arange(n) * 7) % 53
        d = np.uint64(1) + (synth.splitmix64(61, n) >> (64 - bits).astype(np.uint64))
        k = np.cumsum(d, dtype=np.uint64)
    else:
        k = synth.uniform_keys(n, 62, bits=int(kind))
        k[k == M64] = 0
    return np.unique(k)


def probes(keys, head, q, seed):
    edge = np.concatenate([head[head != M64], head[head != M64] - 1, head[head != M64] + 1, keys[:2], keys[-2:],
                           np.array([0, M64, M64 - 1, 1], np.uint64)]).astype(np.uint64)
    pick = keys[synth.splitmix64(seed, q) % np.uint64(len(keys))]
    pick[1::3] += 1
    if q <= len(edge):
        return edge[synth.splitmix64(seed + 1, q) % np.uint64(len(edge))]
    return np.concatenate([edge, pick])[:q]


SETS = [(64, "40", 2000), (128, "dense", 3000), (256, "mixed", 4000), (1024, "40", 60000), (1024, "mixed", 20000),
        (1024, "64", 20000), (2048, "33", 50000), (4096, "40", 100000), (1024, "40", 1)]


@pytest.mark.parametrize("S,kind,n", SETS)
def test_keys(cp, orc, S, kind, n):
    keys = key_set(kind, n)
    for raw in (False, True):
        c = cp.CPMA(keys, leaf_bytes=S, uncompressed=raw)
        head = c.export()[2]
        for q in (1, 3, 4, 5, 64, 65, 20000):
            x = probes(keys, head, q, 6300 + q)
            want = orc.contains(keys, x)
            want[x == M64] = 0
            assert np.array_equal(c.contains(x), want), (raw, q)
            lo, hi = x, probes(keys, head, q, 6400 + q)
            s, m = c.range_map(lo, hi)
            es, em = orc.range_map(keys, lo, hi)
            assert np.array_equal(m, em) and np.array_equal(s, es), (raw, q)
        c.close()


@pytest.mark.parametrize("S,kind,n", [(64, "40", 500), (128, "dense", 3000), (1024, "mixed", 4000), (1024, "40", 20000),
                                      (4096, "64", 30000)])
def test_values(cp, orc, S, kind, n):
    keys = key_set(kind, n)
    vals = synth.uniform_keys(len(keys), 6500, bits=64)
    c = cp.CPMA(keys, leaf_bytes=S, values=vals)
    head = c.export()[2]
    for q in (1, 4, 5, 65, 20000):
        x = probes(keys, head, q, 6600 + q)
        v, f = c.get(x)
        ev, ef = orc.kv_get(keys, vals, x)
        assert np.array_equal(f, ef) and np.array_equal(v, ev), q
        assert np.array_equal(c.contains(x), ef), q
        lo, hi = x, probes(keys, head, q, 6700 + q)
        s, m = c.range_map_values(lo, hi)
        es, em = orc.kv_range_values(keys, vals, lo, hi)
        assert np.array_equal(m, em) and np.array_equal(s, es), q
        s, m = c.range_map(lo, hi)
        es, em = orc.range_map(keys, lo, hi)
        assert np.array_equal(m, em) and np.array_equal(s, es), q
    c.close()
