"""Bottom-up invocations of a relabelled symmetric graph look at a vertex's
first four neighbours in a place of their own and skip the vertices without
edges: rows of zero to nine entries, sources with and without edges, against
the oracle and the plain upload."""
import numpy as np
import pytest

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


def _rows(n, k, isolated):
    """Circulant graph of degree k (k even) on n vertices, then isolated ones."""
    u = [i for i in range(n) for _ in range(k // 2)]
    v = [(i + d) % n for i in range(n) for d in range(1, k // 2 + 1)]
    g = gg.from_edges(n + isolated, u + v, v + u, [1 + i % 7 for i in range(len(u))] * 2)
    g.symmetric = True
    return g


GRAPHS = {f"rows of {k}": (lambda k=k: _rows(3001, k, 77)) for k in (2, 4, 6, 8)}
GRAPHS["no edge at the end"] = lambda: _rows(64, 4, 0)
GRAPHS["one edge"] = lambda: _rows(2, 2, 130)
GRAPHS["rmat 13"] = lambda: gg.rmat(13, 10, seed=2, weight_seed=3)
GRAPHS["uniform"] = lambda: gg.uniform_random(20011, 5.0, seed=4, weight_seed=5)


@pytest.mark.parametrize("name", list(GRAPHS))
def test_bottom_up(irgl, name):
    g = GRAPHS[name]()
    rp, col, w = g.numpy()
    deg = np.diff(rp)
    sources = [int(np.argmax(deg)), int(np.argmin(deg))]
    for reorder in (True, False):
        hg = irgl.upload(g.to("cuda"), reorder=reorder)
        for src in sources:
            ref = oracle.bfs(rp, col, src)[0]
            for cfg in ({"do_alpha": 1000000, "do_beta": 1000000, "grid": 9}, {"do_alpha": 1000000, "grid": 64},
                        {"grid": 3, "block": 256}, None):
                print(f"[case] {name} src={src} reorder={reorder} {cfg}", flush=True)
                out, par, st = irgl.query(hg, irgl.IRGL_KIND_BFS, src, with_parent=True, cfg=cfg)
                np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
                oracle.validate(rp, col, src, ref, par.cpu().numpy())
                assert st["frontier_edges"] == oracle.edges_scanned(rp, ref)
                assert st["items"] == int((ref != oracle.INF).sum())
