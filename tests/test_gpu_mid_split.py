"""Batches of 4097 to 2^18 keys: the split into small buckets, taken when the last
such batch's bit length holds and no bucket overflows, and the radix passes
otherwise.  Sizes at the range's ends and around tiles, repeats, fewer and more
bits, skewed batches (16 radix-sorted batches follow one).  The path is read from
the sort phase's bytes per key (40: split, 24 per pass plus 24: passes); set and
layout against the oracle."""
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


def batch(k, bits, seed, distinct=None):
    """k keys in random order, the highest key of the bit length among them."""
    keys = synth.uniform_keys(distinct or k, seed, bits=bits)
    r = np.random.default_rng(seed)
    keys = keys[r.integers(0, len(keys), k)] if distinct else keys
    keys[r.integers(0, k)] = np.uint64((1 << bits) - 1)
    keys[0] = max(keys[0], np.uint64(2))
    keys[1] = np.uint64(1)  # unsorted
    return keys


def apply(c, S, keys, orc, delete=False):
    c.stats_select(["sort"])
    S, n = (orc.delete if delete else orc.insert)(S, keys)
    assert (c.delete_batch if delete else c.insert_batch)(keys) == n
    per_key = c.stats()["sort"][2] / len(keys)
    c.stats_select([])
    b, u, h = c.export()
    code, msg = orc.check_image(b, u, h, c.geometry()[1], S)
    assert code == 0, msg
    return S, per_key


def start(cp, orc):
    base = synth.uniform_keys(3000, 91, bits=40)  # below the range: prepared without it
    return cp.CPMA(base), orc.build_set(base)


@pytest.mark.parametrize("k", [4097, 8192, 8193, 100_000, (1 << 18) - 1, 1 << 18])
@pytest.mark.parametrize("distinct", [None, 300])
def test_sizes(cp, orc, k, distinct):
    print(f"[mid split] k={k} distinct={distinct}", flush=True)
    c, S = start(cp, orc)
    S, per_key = apply(c, S, batch(k, 40, 92, distinct), orc)
    assert per_key == 144
    S, per_key = apply(c, S, batch(k, 40, 93, distinct), orc)
    # a few hundred keys repeated: their buckets may overflow
    assert per_key == 40 or (distinct and per_key == 144)
    S, per_key = apply(c, S, batch(k, 40, 94), orc, delete=True)
    S, per_key = apply(c, S, np.concatenate([S[::3], batch(4097, 40, 95)])[: 1 << 18], orc, delete=True)
    c.close()


def test_bit_lengths(cp, orc):
    c, S = start(cp, orc)
    lsd = {bits: 24 * ((bits + 7) // 8) + 24 for bits in (39, 40, 41)}
    for step, (k, bits, want) in enumerate([
            (9000, 40, lsd[40]), (9000, 40, 40), (9000, 39, 40),   # fewer bits: the counts hold
            (9000, 40, lsd[40]),                                   # more bits than the last batch
            (9000, 40, 40), (9000, 41, lsd[41]), (9000, 41, lsd[41]),  # a low part of 33 bits
            (9000, 40, lsd[40]), (9000, 40, 40),
    ]):
        print(f"[mid split] step {step} bits={bits}", flush=True)
        S, per_key = apply(c, S, batch(k, bits, 100 + step), orc)
        assert per_key == want, step
    c.close()


def test_skewed(cp, orc):
    """A batch that crowds one bucket falls back, the next 16 do not try."""
    c, S = start(cp, orc)
    S, _ = apply(c, S, batch(20000, 40, 110), orc)
    S, per_key = apply(c, S, batch(20000, 40, 111), orc)
    assert per_key == 40
    crowd = batch(20000, 20, 112)
    crowd[5] = np.uint64((1 << 40) - 1)
    S, per_key = apply(c, S, crowd, orc)
    assert per_key == 144
    paths = []
    for i in range(18):
        S, per_key = apply(c, S, batch(5000, 40, 120 + i), orc)
        paths.append(per_key)
    assert paths == [144] * 16 + [40, 40], paths
    c.close()
