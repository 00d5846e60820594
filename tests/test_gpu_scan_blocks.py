"""Prefix sums around 1024 blocks of 2048 items, where the apply blocks stop adding
the totals up themselves: key-value batches (one flag per key), spread over the
whole key space with repeats.  Counts, and the value of every key, exact."""
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


@pytest.mark.parametrize("k", [2048, 2049, (1 << 21) - 2047, 1 << 21, (1 << 21) + 1, (1 << 21) + 2049])
def test_flags(cp, k):
    print(f"[scan blocks] k={k}", flush=True)
    keys = synth.uniform_keys(k, 81, bits=40)
    keys[1::3] = keys[::3][: len(keys[1::3])]
    vals = synth.uniform_keys(k, 82, bits=64)
    c = cp.CPMA(np.arange(5, dtype=np.uint64), values=np.zeros(5, np.uint64))
    uniq, first = np.unique(keys, return_index=True)
    new = int(np.sum(uniq >= 5))
    assert c.insert_kv(keys, vals) == new
    got, found = c.get(uniq)
    assert np.all(found) and np.array_equal(got, vals[first])
    c.close()
