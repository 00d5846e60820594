"""Batch merges by splices: inserts before heads, behind last keys and in every
gap, up to 64 per leaf and into overflow; deletes of single keys, runs, heads,
tails, whole leaves and every second key (more than 64 splices in a leaf), with
absent keys among them; codes of 1 to 5 bytes, leaves from 64 to 1024 bytes.
Exact against the oracle, the layout through the structure checker."""
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


def check(c, expect, orc):
    b, u, h = c.export()
    code, msg = orc.check_image(b, u, h, c.geometry()[1], expect)
    assert code == 0, msg
    assert c.size() == len(expect)


def insert(c, expect, keys, orc):
    expect, added = orc.insert(expect, keys)
    assert c.insert_batch(keys) == added
    check(c, expect, orc)
    return expect


def delete(c, expect, keys, orc):
    expect, removed = orc.delete(expect, keys)
    assert c.delete_batch(keys) == removed
    check(c, expect, orc)
    return expect


@pytest.mark.parametrize("S", [64, 512, 1024])
@pytest.mark.parametrize("gap", [1, 3, 100, 20000, 3000000, 400000000])
def test_splices(cp, orc, S, gap):
    """Gaps of 1 to 400000000 between keys: codes of 1 to 5 bytes."""
    n = 60000
    r = np.random.default_rng(gap)
    steps = r.integers(1, 2 * gap, n).astype(np.uint64) if gap > 1 else np.ones(n, np.uint64)
    base = np.cumsum(steps) + np.uint64(10**7)
    cfg = cp.default_config()
    cfg.leaf_bytes, cfg.rebuild_frac = S, 10.0
    c = cp.CPMA(base, config=cfg)
    expect = base
    heads = c.export()[2]
    print(f"[splices] S={S} gap={gap} leaves={len(heads)}", flush=True)
    heads = heads[heads != np.uint64(2**64 - 1)]
    # every second key, then runs around every head, then the lot back
    expect = delete(c, expect, np.concatenate([base[::2], base[1::2] + np.uint64(1)]), orc)
    expect = insert(c, expect, base, orc)
    pos = np.searchsorted(base, heads)
    runs = np.unique(np.clip((pos[:, None] + np.arange(-3, 4)[None, :]).ravel(), 0, n - 1))
    expect = delete(c, expect, np.concatenate([base[runs], base[: 5000]]), orc)
    # below every head, behind every leaf's last key, in random gaps
    near = np.concatenate([heads - np.uint64(1), heads - np.uint64(2), heads + np.uint64(1)])
    more = base[r.integers(0, n, 9000)] + r.integers(0, 2 * gap, 9000).astype(np.uint64)
    expect = insert(c, expect, np.concatenate([near, more, base[runs]]), orc)
    # up to 64 keys around one key of many leaves: overflow
    at = base[r.integers(0, n, 200)][:, None] + np.arange(60, dtype=np.uint64)[None, :]
    expect = insert(c, expect, at.ravel(), orc)
    # whole leaves, then nearly everything
    expect = delete(c, expect, expect[3000:9000], orc)
    keep = r.random(len(expect)) < 0.02
    expect = delete(c, expect, expect[~keep], orc)
    expect = insert(c, expect, base[::3], orc)
    c.close()
