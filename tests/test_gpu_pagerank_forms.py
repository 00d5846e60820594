"""PageRank on graphs around the rules that choose between the binned form and the pull
with 64-bit sums, and the pull of sparse graphs: one set, few and many iterations,
hubs whose edges fill leaves, ids beyond nv.  Error against FP64 ranks; the two forms
that sum in 64 bits differ by their contributions' rounding only."""
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


@pytest.mark.parametrize("nv,m,skew", [(1 << 12, 40_000, False), (1 << 16, 400_000, True), (1 << 18, 1_000_000, False),
                                       (1 << 20, 500_000, False), (1 << 20, 1_000_000, True), (1 << 21, 300_000, False)])
@pytest.mark.parametrize("iters", [1, 2, 9, 20])
def test_forms(cp, orc, nv, m, skew, iters):
    src, dst = synth.er_edges(m, 8300 + m, nv)
    if skew:
        src = (src * src) // np.uint64(nv)
        src[: m // 10] = 7  # a hub whose edges fill many leaves
    keys = np.unique(synth.edge_keys(src, dst, symmetric=True))
    c = cp.CPMA(keys)
    want = orc.pagerank(keys, nv, iters=iters)
    got = c.pagerank(nv, iters=iters).astype(np.float64)
    # 32-bit contributions: each step's relative rounding is a few 2^-24
    assert np.max(np.abs(got - want) / want) < 2e-6 + 4e-7 * iters
    half = nv // 2 + 1
    ok = ((keys >> np.uint64(32)) < half) & ((keys & np.uint64(0xffffffff)) < half)
    want = orc.pagerank(keys[ok], half, iters=iters)
    got = c.pagerank(half, iters=iters).astype(np.float64)
    assert np.max(np.abs(got - want) / want) < 2e-6 + 4e-7 * iters
    c.close()
