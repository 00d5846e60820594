"""Whole leaves whose keys span 2^32 and more, in scans of range_map: codes of one to
ten bytes that fall on both sides of a leaf's halves, next to leaves of smaller spans;
leaf by leaf and through the prefix sums of many queries; keys of plain and key-value
sets.  Against the oracle."""
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


def mixed_keys(n, seed, widest):
    """n keys whose deltas take 1 to `widest` bits, in runs of 40 of one width, short ones more often."""
    r = np.random.default_rng(seed)
    bits = np.repeat(np.where(r.random(n // 40 + 1) < 0.6, r.integers(1, 33, n // 40 + 1),
                              r.integers(1, widest + 1, n // 40 + 1)), 40)[:n]
    deltas = [int(x) % (1 << int(b)) + 1 for x, b in zip(r.integers(0, 1 << 62, n), bits)]
    keys, at = [], 0
    for d in deltas:
        if at + d >= (1 << 64) - 2:
            break
        at += d
        keys.append(at)
    return np.array(keys, np.uint64)


@pytest.mark.parametrize("S", [64, 256, 1024, 4096])
@pytest.mark.parametrize("widest", [34, 52, 57])
@pytest.mark.parametrize("values", [False, True])
def test_scans(cp, orc, S, widest, values):
    for seed in range(2):
        keys = mixed_keys(60000, 7950 + seed, widest)
        c = cp.CPMA(keys, leaf_bytes=S, values=keys if values else None)
        _, _, head = c.export()
        r = np.random.default_rng(7960 + seed)
        for q in (1, 3, 200):  # 200 whole scans: through the prefix sums
            lo = np.zeros(q, np.uint64)
            hi = np.full(q, (1 << 64) - 1, np.uint64)
            if q == 200:  # every second range starts and ends at heads and beside them
                i = np.sort(r.integers(0, len(head), (100, 2)), axis=1)
                lo[::2], hi[::2] = head[i[:, 0]], head[i[:, 1]] + r.integers(0, 2, 100).astype(np.uint64)
            s, n = c.range_map(lo, hi)
            es, en = orc.range_map(keys, lo, hi)
            assert np.array_equal(n, en) and np.array_equal(s, es), (seed, q)
        c.close()


def test_ten_byte_codes(cp, orc):
    """Keys 2^62 and more apart, a few in each leaf of otherwise dense keys."""
    dense = np.arange(0, 40000, dtype=np.uint64)
    top = (1 << 64) - 2
    keys = np.concatenate([dense, np.array([1 << 62, (1 << 62) + 1, 1 << 63, top - 1, top], np.uint64)])
    far = np.concatenate([np.array([0, 1], np.uint64), np.arange(top - 3000, top, 3, dtype=np.uint64)])
    for k in (keys, far):
        for S in (64, 128, 1024, 4096):
            c = cp.CPMA(k, leaf_bytes=S)
            lo, hi = np.array([0, 0, 1, 5], np.uint64), np.array([top + 1, top, 1 << 63, top], np.uint64)
            s, n = c.range_map(lo, hi)
            es, en = orc.range_map(k, lo, hi)
            assert np.array_equal(n, en) and np.array_equal(s, es), S
            c.close()


@pytest.mark.parametrize("S", [64, 1024, 4096])
@pytest.mark.parametrize("values", [False, True])
def test_lookups_over_mixed_leaves(cp, orc, S, values):
    """Lookups of one wave in leaves of small and of wide spans, beside and at their keys."""
    keys = mixed_keys(40000, 7970, 52)
    c = cp.CPMA(keys, leaf_bytes=S, values=keys if values else None)
    r = np.random.default_rng(7971)
    at = keys[r.integers(0, len(keys), 6000)]
    x = at + r.integers(0, 3, 6000).astype(np.uint64) - np.uint64(1)
    width = np.uint64(1) << r.integers(0, 60, 6000).astype(np.uint64)
    hi = np.minimum(x, np.uint64((1 << 64) - 2) - width) + width
    for sel in (slice(None), slice(0, 7)):
        s, n = c.range_map(x[sel], hi[sel])
        es, en = orc.range_map(keys, x[sel], hi[sel])
        assert np.array_equal(n, en) and np.array_equal(s, es)
        assert np.array_equal(c.contains(x[sel]), orc.contains(keys, x[sel]))
        if values:
            v, found = c.get(x[sel])
            member = orc.contains(keys, x[sel]).astype(bool)
            assert np.array_equal(found.astype(bool), member)
            assert np.array_equal(v, np.where(member, x[sel], np.uint64(0)))
    c.close()
