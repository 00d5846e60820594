"""The fused pass's item passes and per-leaf membership: empty, tiny and large
requests mixed (the gather and the kind bytes divide positions, not requests),
from host and from device memory, on leaves within 2^32 and beyond, of 512 to
2048 bytes.  Counts and final set against the oracle replaying the requests."""
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


SIZES = {
    "mixed": [0, 1, 0, 0, 70001, 0, 3, 17, 1023, 1024, 1025, 0, 30000, 2, 0],
    "tiny": [1, 0, 2, 0] * 3000,
    "odd_total": [4097],
}


@pytest.mark.parametrize("device", [False, True])
@pytest.mark.parametrize("sizes", list(SIZES))
@pytest.mark.parametrize("bits,S", [(22, 1024), (40, 512), (64, 1024), (40, 2048), (64, 2048)])
def test_requests(cp, orc, bits, S, sizes, device):
    import torch
    print(f"[fused routes] bits={bits} S={S} {sizes} device={device}", flush=True)
    base = np.unique(synth.uniform_keys(20000, 61, bits=bits))
    c = cp.CPMA(base, leaf_bytes=S)
    expect, reqs, counts = base, [], []
    for i, n in enumerate(SIZES[sizes]):
        keys = synth.uniform_keys(n, 62 + i, bits=bits)
        keys[::2] = base[synth.uniform_keys(len(keys[::2]), 63 + i, bits=14).astype(np.int64)]
        if i % 3 == 2:
            expect, cnt = orc.delete(expect, keys)
            reqs.append((cp.REQ_DELETE, keys))
        else:
            expect, cnt = orc.insert(expect, keys)
            reqs.append((cp.REQ_INSERT, keys))
        counts.append(cnt)
    if device:
        reqs = [(kind, torch.from_numpy(k.view(np.int64)).cuda()) for kind, k in reqs]
    assert c.apply_updates(reqs) == counts
    b, u, h = c.export()
    code, msg = orc.check_image(b, u, h, c.geometry()[1], expect)
    assert code == 0, msg
    assert c.size() == len(expect)
