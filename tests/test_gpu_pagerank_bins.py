"""PageRank over binned edges: vertex counts around the parts' and bins' sizes,
hubs, vertices without edges, directed edge sets, edges to vertices beyond nv, and
edge counts on both sides of the rule that chooses the binned form.  Within 1e-5
of FP64 ranks (the oracle's; for directed sets the pull form written out here)."""
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


def edge_set(kind, nv, m):
    if kind == "star":
        d = np.arange(1, nv, dtype=np.uint64)
        return np.unique(np.concatenate([d, d << np.uint64(32)]))
    src, dst = synth.er_edges(m, 8100 + m, nv)
    if kind == "skew":  # most edges from and to the lowest ids
        src, dst = (src * src) // np.uint64(nv), (dst * dst * dst) // np.uint64(nv * nv)
    return np.unique(synth.edge_keys(src, dst, symmetric=kind != "directed"))


def pull(keys, nv, iters):
    """FP64 ranks in pull form: u sums p[v] / deg[v] over its edges (u, v), which on a
    directed set is not the push form of the oracle."""
    src, dst = (keys >> np.uint64(32)).astype(np.int64), (keys & np.uint64(0xffffffff)).astype(np.int64)
    deg = np.bincount(src, minlength=nv)
    p = np.full(nv, 1.0 / nv)
    for _ in range(iters):
        share = np.where(deg > 0, p / np.maximum(deg, 1), 0.0)
        p = 0.15 / nv + 0.85 * np.bincount(src, weights=share[dst], minlength=nv)
    return p


def check(cp, orc, keys, nv, iters, symmetric=True):
    c = cp.CPMA(keys)
    got = c.pagerank(nv, iters=iters).astype(np.float64)
    ok = ((keys >> np.uint64(32)) < nv) & ((keys & np.uint64(0xffffffff)) < nv)
    want = orc.pagerank(keys[ok], nv, iters=iters) if symmetric else pull(keys[ok], nv, iters)
    assert np.max(np.abs(got - want) / want) < 1e-5
    again = c.pagerank(nv, iters=iters)
    assert np.max(np.abs(again - want) / want) < 1e-5
    c.close()


@pytest.mark.parametrize("kind", ["uniform", "skew", "directed"])
@pytest.mark.parametrize("nv,m", [(1, 10), (100, 20000), (32768, 300000), (32769, 300000), (65537, 20000),
                                  (131071, 600000), (300001, 3000000)])
def test_sizes(cp, orc, kind, nv, m):
    keys = edge_set(kind, nv, m) if nv > 1 else np.array([0], np.uint64)
    for iters in (0, 1, 4):
        check(cp, orc, keys, nv, iters, kind != "directed")


def test_star(cp, orc):
    check(cp, orc, edge_set("star", 400000, 0), 400000, 3)


def test_ids_beyond_nv(cp, orc):
    keys = edge_set("uniform", 200000, 2000000)
    for nv in (150001, 8192):
        check(cp, orc, keys, nv, 2)
