"""BFS levels, top-down and bottom-up, on graphs that reach every form of the
step: sources close together and thousands of ids apart inside one lane, hubs
that fill whole leaves, long paths (many bottom-up levels, most leaves done
early), vertices without edges, ids at and past nv, nv at and around multiples
of 32.  Exact against the oracle."""
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


def edge_keys(u, v):
    u, v = np.concatenate([u, v]).astype(np.uint64), np.concatenate([v, u]).astype(np.uint64)
    return np.unique((u << np.uint64(32)) | v)


def graph(name):
    r = np.random.default_rng(17)
    if name == "sparse_ids":      # ids 1000 apart: no two sources share a word
        return r.integers(0, 3000, 9000) * 1000, r.integers(0, 3000, 9000) * 1000, 3000 * 1000 + 5
    if name == "one_edge_each":   # many sources per lane, ids 3 apart
        n = 60000
        p = r.permutation(n) * 3
        return p[: n // 2], p[n // 2:], 3 * n
    if name == "low_degree":      # several bottom-up levels, isolated vertices
        return r.integers(0, 40000, 70000) * 2, r.integers(0, 40000, 70000) * 2, 80000
    if name == "hub_and_tails":
        hub = np.zeros(50000, np.int64), np.arange(1, 50001)
        tail = np.arange(1, 50001), np.arange(50001, 100001)
        far = np.arange(50001, 100000), np.arange(50002, 100001)
        parts = [hub, tail, (far[0][::7], far[1][::7])]
        return np.concatenate([x[0] for x in parts]), np.concatenate([x[1] for x in parts]), 100001
    u = r.integers(0, 20000, 400000)  # dense: one level reaches most
    return u, r.integers(0, 20000, 400000), 20000


@pytest.mark.parametrize("S", [64, 1024])
@pytest.mark.parametrize("name", ["sparse_ids", "one_edge_each", "low_degree", "hub_and_tails", "dense"])
def test_levels(cp, orc, name, S):
    u, v, n = graph(name)
    keys = edge_keys(u, v)
    c = cp.CPMA(keys, leaf_bytes=S)
    for nv in (n, n + 31, (n + 31) // 32 * 32, n - n // 3):
        src = int(u[u < nv][0])
        print(f"[bfs] {name} S={S} nv={nv} src={src}", flush=True)
        inside = keys[((keys >> np.uint64(32)) < nv) & ((keys & np.uint64(0xFFFFFFFF)) < nv)]
        want = orc.bfs(inside, nv, src)
        assert np.array_equal(c.bfs(nv, src, symmetric=True), want)
        assert np.array_equal(c.bfs(nv, src), want)
    c.close()
