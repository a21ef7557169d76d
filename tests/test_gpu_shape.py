"""The default launch shape of single queries, at the entry counts where it
changes: results do not depend on it, and an explicit grid is kept."""
import numpy as np
import pytest

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu

BFS, SSSP = 0, 1


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


def _cut(g, m):
    """The first m / 2 undirected edges of a symmetric graph."""
    rp, col, w = g.numpy()
    s = np.repeat(np.arange(g.n), np.diff(rp))
    keep = np.nonzero(s < col)[0][:m // 2]
    u, v, x = s[keep].tolist(), col[keep].tolist(), w[keep].tolist()
    out = gg.from_edges(g.n, u + v, v + u, x + x)
    out.symmetric = True
    return out


@pytest.mark.parametrize("m,workgroups", [
    (8190, (1, 1)), (8194, (1, 128)), (16384, (1, 128)), (65536, (1, 128)), (65538, (64, 128)),
])
def test_uniform_graphs(irgl, m, workgroups):
    g = _cut(gg.uniform_random(1000, 80.0, seed=3, weight_seed=4), m)
    assert g.m == m
    rp, col, w = g.numpy()
    hg = irgl.upload(g.to("cuda"))
    src = gg.pick_sources(g, 1, seed=5)[0]
    refs = (oracle.bfs(rp, col, src)[0], oracle.dijkstra(rp, col, w, src)[0])
    for kind in (BFS, SSSP):
        print(f"[case] m={m} kind={kind}", flush=True)
        for cfg in (None, {"grid": 5}, {"block": 256}):
            out, _, st = irgl.query(hg, kind, src, with_parent=True, cfg=cfg)
            np.testing.assert_array_equal(irgl.as_u32_numpy(out), refs[kind])
            if cfg is None:
                assert st["grid"] == workgroups[kind]
            elif "grid" in cfg:
                assert st["grid"] == 5


@pytest.mark.parametrize("make,kinds", [
    (lambda: gg.rmat(17, 12, seed=1, weight_seed=2), (128, 256)),
    (lambda: gg.uniform_random(70000, 14.9, seed=1, weight_seed=2), (64, 128)),
    (lambda: gg.uniform_random(70000, 15.1, seed=1, weight_seed=2), (128, 256)),
    (lambda: gg.random_directed(70000, 1 << 20, seed=1, weight_seed=2), (128, 128)),
    (lambda: gg.random_directed(70000, (1 << 20) + 1, seed=1, weight_seed=2), (256, 256)),
])
def test_larger_graphs(irgl, make, kinds):
    g = make()
    rp, col, w = g.numpy()
    for reorder in (False, True):
        hg = irgl.upload(g.to("cuda"), reorder=reorder)
        src = gg.pick_sources(g, 1, seed=5)[0]
        for kind in (BFS, SSSP):
            print(f"[case] {g.name} kind={kind} reorder={reorder}", flush=True)
            out, _, st = irgl.query(hg, kind, src)
            ref = oracle.bfs(rp, col, src)[0] if kind == BFS else oracle.dijkstra(rp, col, w, src)[0]
            np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
            if not reorder:
                assert st["grid"] == kinds[kind]
