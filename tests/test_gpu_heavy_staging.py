"""Long insert slices into leaves above 1 KiB, whose merged keys are staged in memory:
many dense leaves that each take a few hundred keys, on a set whose scratch was
given back.  Staging is reserved before the batch writes, so too little of it breaks
the update.  Counts against the oracle, the layout through the structure checker."""
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


@pytest.mark.parametrize("S", [1024, 2048, 4096])
@pytest.mark.parametrize("per", [257, 300, 400])
@pytest.mark.parametrize("leaves", [4, 10, 13, 200])  # small batches (up to 4096 keys) and ordinary ones
def test_dense_leaves(cp, orc, S, per, leaves):
    keys = np.arange(0, 2 * 700000, 2, dtype=np.uint64)  # one-byte codes
    c = cp.CPMA(keys, leaf_bytes=S)
    c.trim()
    _, used, head = c.export()
    nl = len(head)
    assert nl > leaves
    batch = []
    for i in range(leaves):
        f = i * (nl - 1) // leaves
        first, count = int(head[f]), int(used[f]) - 7
        take = min(per, count - 1)
        batch.append(np.uint64(first + 1) + 2 * synth.sample_indices(count - 1, take, 7700 + i).astype(np.uint64))
    batch = np.concatenate(batch)
    expect, added = orc.insert(keys, batch)
    assert c.insert_batch(batch) == added
    b, u, h = c.export()
    code, msg = orc.check_image(b, u, h, S, expect)
    assert code == 0, msg
    c.close()
