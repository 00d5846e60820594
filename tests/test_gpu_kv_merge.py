"""The key-value merge's edges: codes of 9 and 10 bytes (keys spread over 64
bits), leaves of more than 64 and 128 keys, slices of more than 64 keys, merged
leaves beyond the LDS room, empty leaves, upserts with and without values.
Layout and contents against the oracle after every batch."""
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


def check(c, K, V, orc):
    b, u, h = c.export()
    code, msg = orc.check_image_kv(b, u, c.code_bytes(), h, c.geometry()[1], K, V)
    assert code == 0, msg
    got, found = c.get(K)
    assert np.all(found) and np.array_equal(got, V)


def vals(keys, seed):
    return synth.uniform_keys(len(keys), seed, bits=64)


@pytest.mark.parametrize("S", [64, 1024, 4096])
@pytest.mark.parametrize("bits,n", [(64, 3), (64, 40), (64, 3000), (12, 3000), (40, 30000)])
def test_merge(cp, orc, S, bits, n):
    print(f"[kv merge] S={S} bits={bits} n={n}", flush=True)
    base = np.unique(synth.uniform_keys(n, 31, bits=bits))
    c = cp.CPMA(base, leaf_bytes=S, values=vals(base, 32))
    K, V = orc.kv_build(base, vals(base, 32))
    for step, k in enumerate((7, 63, 65, 900, 3 * n + 200)):
        keys = np.concatenate([synth.uniform_keys(k, 40 + step, bits=bits), base[:: step + 2],
                               np.array([0, 1, (1 << min(bits, 63)) - 1], np.uint64)])
        v = vals(keys, 50 + step)
        K, V, added = orc.kv_insert(K, V, keys, v)
        assert c.insert_kv(keys, v) == added
        check(c, K, V, orc)
        gone = np.concatenate([K[step::3], keys[:20]])
        K, V, removed = orc.kv_delete(K, V, gone)
        assert c.delete_batch(gone) == removed
        check(c, K, V, orc)
        kept = V.copy()
        assert c.insert_batch(K[::2]) == 0  # present keys without values keep theirs
        check(c, K, kept, orc)
