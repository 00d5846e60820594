"""The radix passes' tiles: sizes on both sides of the small tile's limit
(393216 keys), of the tile count up to which a scatter block adds up the other
tiles' counts itself (384 tiles of 4096 keys), ragged last tiles and batches
full of repeats (one digit holds a whole tile).  64-bit keys keep the larger
batches out of the split into buckets.  Exact against the oracle."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu

SMALL = 3 << 17
SUMS = 384 * 4096
SIZES = [4097, 5000, SMALL - 1, SMALL, SMALL + 1, SUMS, SUMS + 1, SUMS + 4097]


@pytest.fixture(scope="module")
def cp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2305_05055_amd as p
    p.lib()
    return p


def batch(k, seed, distinct):
    pool = synth.unique_uniform_keys(distinct, seed, bits=64)
    pool = pool[pool != np.uint64(0xFFFFFFFFFFFFFFFF)]
    return pool[np.random.default_rng(seed).integers(0, len(pool), k)]


@pytest.mark.parametrize("k", SIZES)
@pytest.mark.parametrize("repeats", [1, 500])
def test_keys(cp, orc, k, repeats):
    print(f"[sort tiles] keys k={k} repeats={repeats}", flush=True)
    keys = batch(k, 700 + k % 97, max(8, k // repeats))
    c = cp.CPMA(synth.uniform_keys(5000, 3, bits=64))
    S = orc.build_set(synth.uniform_keys(5000, 3, bits=64))
    S, added = orc.insert(S, keys)
    assert c.insert_batch(keys) == added
    b, u, h = c.export()
    code, msg = orc.check_image(b, u, h, c.geometry()[1], S)
    assert code == 0, msg
    asc = np.sort(batch(k, 900 + k % 89, max(8, k // repeats)))  # sorted: only repeats are removed
    S, added = orc.insert(S, asc)
    assert c.insert_batch(asc) == added
    assert c.size() == len(S)
    assert c.range_map(np.array([0], np.uint64), np.array([2**64 - 1], np.uint64))[1][0] == len(S)


@pytest.mark.parametrize("k", SIZES)
def test_values(cp, k):
    """The value of a repeated key is its first occurrence's."""
    print(f"[sort tiles] values k={k}", flush=True)
    keys = batch(k, 800 + k % 97, max(8, k // 3))
    vals = synth.uniform_keys(k, 801, bits=64)
    c = cp.CPMA(np.zeros(0, np.uint64), values=np.zeros(0, np.uint64))
    uniq, first = np.unique(keys, return_index=True)
    assert c.insert_kv(keys, vals) == len(uniq)
    got, found = c.get(uniq)
    assert np.all(found)
    assert np.array_equal(got, vals[first])


def test_skewed_batches_in_a_row(cp, orc):
    """A second skewed batch of the same bit length goes to the radix passes after
    one count of its buckets; the batches after it are split again."""
    c = cp.CPMA(synth.uniform_keys(50000, 5, bits=34))
    S = orc.build_set(synth.uniform_keys(50000, 5, bits=34))
    r = np.random.default_rng(9)
    top = np.uint64((1 << 34) - 1)  # every batch has the same bit length
    for i, kind in enumerate("zzuzu"):
        keys = synth.zipf_keys(600_000, 6 + i, bits=34) if kind == "z" else synth.uniform_keys(600_000, 6 + i, bits=34)
        keys = np.concatenate([keys, [top]])[r.permutation(len(keys) + 1)]
        print(f"[sort tiles] batch {i} {kind}", flush=True)
        c.stats_select(["sort"])
        S, added = orc.insert(S, keys)
        assert c.insert_batch(keys) == added
        assert c.stats()["sort"][2] / len(keys) == (144 if kind == "z" else 40), (i, kind)
        c.stats_select([])
        b, u, h = c.export()
        code, msg = orc.check_image(b, u, h, c.geometry()[1], S)
        assert code == 0, msg
