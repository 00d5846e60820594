"""Insert slices of more than 4096 keys, which are merged piece by piece: sizes
around the piece and giant limits, old keys below, between and above the batch,
batch keys already present, several giants in one batch, and with a rebuild.
Counts against the oracle, the layout through the structure checker."""
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
    L, S = c.geometry()
    code, msg = orc.check_image(b, u, h, S, expect)
    assert code == 0, msg
    assert c.size() == len(expect)


def run(c, expect, batch, orc):
    expect, added = orc.insert(expect, batch)
    assert c.insert_batch(batch) == added
    check(c, expect, orc)
    expect, removed = orc.delete(expect, batch[::2])
    assert c.delete_batch(batch[::2]) == removed
    check(c, expect, orc)
    return expect


@pytest.mark.parametrize("S", [64, 1024, 4096])
@pytest.mark.parametrize("k", [4096, 4097, 5120, 5121, 9000, 60001])
def test_one_leaf(cp, orc, S, k):
    """k keys in one gap of the set, with the gap's own neighbours among them."""
    keys = orc.build_set(synth.uniform_keys(20000, 7100, bits=40) | np.uint64(1 << 39))
    for at in (0, 10007, len(keys) - 1):  # below every key, inside, above
        c = cp.CPMA(keys, leaf_bytes=S)
        base = int(keys[at])
        lo = base - 2 * k if at == 0 else base + 1
        batch = np.uint64(lo) + synth.sample_indices(8 * k, k, 7200 + k).astype(np.uint64)
        batch[:50] = keys[max(0, at - 60):][:50] if len(keys) - max(0, at - 60) >= 50 else keys[-50:]
        run(c, keys, batch, orc)
        c.close()


@pytest.mark.parametrize("S,rebuild", [(1024, 1.0), (1024, 0.01), (256, 1.0), (2048, 1.0)])
def test_several(cp, orc, S, rebuild):
    keys = orc.build_set(synth.uniform_keys(50000, 7300, bits=40))
    cfg = cp.default_config()
    cfg.leaf_bytes, cfg.rebuild_frac = S, rebuild
    c = cp.CPMA(keys, config=cfg)
    parts = [keys[i] + np.arange(1, 2 + 3 * k, 3, dtype=np.uint64) for i, k in
             ((3, 5000), (1000, 4097), (20000, 70000), (20400, 300), (49999, 6000))]
    batch = np.concatenate(parts + [synth.uniform_keys(30000, 7301, bits=40), keys[::11]])
    batch = batch[synth.splitmix64(7302, len(batch)).argsort()]
    expect = run(c, keys, batch, orc)
    run(c, expect, np.concatenate(parts)[::-1] + np.uint64(1), orc)
    c.close()


@pytest.mark.parametrize("k", [20000, 100000])
def test_wide_keys(cp, orc, k):
    """Keys above 2^53: the code at a piece's start counts from the exact key
    before it, an old key or a batch key."""
    keys = orc.build_set(synth.uniform_keys(5000, 7400, bits=63))
    c = cp.CPMA(keys)
    run(c, keys, synth.uniform_keys(k, 7401, bits=64), orc)
    c.close()
