"""Interior scans of range_map on either side of the visits from which on a leaf gets one
lane instead of two: through visits leaf by leaf (fewer than 32 queries) and through
the prefix sums, at leaf sizes with different limits, with narrow, wide and mixed
spans, on plain, key-value and raw leaves.  Against prefix sums over the keys."""
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


def expected(keys, sums, lo, hi):
    i, j = np.searchsorted(keys, lo), np.searchsorted(keys, hi)
    j = np.maximum(i, j)
    return sums[j] - sums[i], (j - i).astype(np.uint64)


def check(c, keys, weights, lo, hi, fn):
    sums = np.concatenate([np.zeros(1, np.uint64), np.cumsum(weights, dtype=np.uint64)])
    es, en = expected(keys, sums, lo, hi)
    s, n = fn(lo, hi)
    assert np.array_equal(n, en) and np.array_equal(s, es)


@pytest.mark.parametrize("S,n,bits,form", [
    (64, 150_000, 40, "plain"), (64, 400_000, 63, "plain"), (128, 500_000, 40, "plain"), (256, 900_000, 63, "plain"),
    (512, 1_000_000, 30, "plain"), (1024, 1_000_000, 40, "plain"), (1024, 1_000_000, 24, "plain"),
    (4096, 1_000_000, 40, "plain"), (256, 300_000, 40, "values"), (1024, 900_000, 63, "values"),
    (256, 300_000, 40, "raw"), (1024, 600_000, 40, "raw"),
])
def test_scans(cp, S, n, bits, form):
    keys = np.unique(synth.uniform_keys(n, 8100, bits=bits) % np.uint64((1 << 64) - 2))
    vals = synth.uniform_keys(len(keys), 8101, bits=64) if form == "values" else None
    c = cp.CPMA(keys, leaf_bytes=S, uncompressed=form == "raw", values=vals)
    r = np.random.default_rng(8102)
    for q in (1, 9, 31, 40, 1023, 1024, 1025, 3000):  # blocks scan up to 1024 queries themselves
        a = r.integers(0, len(keys), (q, 2))
        if q <= 40:  # long ranges, so that few queries make many visits
            a[:, 0] //= 50
            a[:, 1] = len(keys) - 1 - a[:, 1] // 50
        a.sort(axis=1)
        lo, hi = keys[a[:, 0]], keys[a[:, 1]] + np.uint64(1)
        lo[0] = 0
        check(c, keys, keys, lo, hi, c.range_map)
        if vals is not None:
            check(c, keys, vals, lo, hi, c.range_map_values)
    c.close()


def test_prefix_over_many_leaves(cp):
    """Prefix sums of more leaves than the limit at 1 KiB, whose last group of 64 is not full."""
    keys = np.unique(synth.uniform_keys(21_000_000, 8103, bits=40))
    c = cp.CPMA(keys)
    assert c.geometry()[0] >= 65536
    a = np.random.default_rng(8104).integers(0, len(keys), (500, 2))
    a.sort(axis=1)
    check(c, keys, keys, keys[a[:, 0]], keys[a[:, 1]], c.range_map)
    c.close()
