"""Which small graphs' queries run on one workgroup: a BFS that stays top-down
only up to 16,384 entries unless no row is longer than 8, a long row never
alone; and worklists just above one item per wavefront, whose tiles are spread
over the team.  Results are the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu

BFS, SSSP = 0, 1
OFF = 0xFFFFFFFF


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


def _star(leaves):
    i = list(range(1, leaves + 1))
    g = gg.from_edges(leaves + 1, [0] * leaves + i, i + [0] * leaves, [1 + x % 50 for x in i] * 2)
    g.symmetric = True
    return g


def _ring(n, k):
    """Every vertex has edges to the next k: n * k entries, no row longer than k."""
    u = [i for i in range(n) for _ in range(k)]
    return gg.from_edges(n, u, [(i + d) % n for i in range(n) for d in range(1, k + 1)], [1 + i % 7 for i in range(n * k)])


def _check(irgl, g, kind, src, cfg=None):
    rp, col, w = g.numpy()
    hg = irgl.upload(g.to("cuda"))
    out, _, st = irgl.query(hg, kind, src, cfg=cfg)
    ref = oracle.bfs(rp, col, src)[0] if kind == BFS else oracle.dijkstra(rp, col, w, src)[0]
    np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
    return st


@pytest.mark.parametrize("make,kind,cfg,one", [
    (lambda: _ring(1024, 16), BFS, None, True),      # 16,384 entries
    (lambda: _ring(1025, 16), BFS, None, False),
    (lambda: _ring(8192, 8), BFS, None, True),       # rows of at most 8: up to 65,536
    (lambda: _ring(7000, 9), BFS, None, False),
    (lambda: gg.uniform_random(8000, 7.9, seed=3, weight_seed=4), BFS, None, True),  # may go bottom-up
    (lambda: gg.uniform_random(8000, 7.9, seed=3, weight_seed=4), BFS, {"do_alpha": OFF}, False),
    (lambda: _star(4096), SSSP, None, True),
    (lambda: _star(4097), SSSP, None, False),
    (lambda: _star(4097), BFS, None, True),
    (lambda: _star(4097), BFS, {"do_alpha": OFF}, False),
])
def test_one_workgroup(irgl, make, kind, cfg, one):
    st = _check(irgl, make(), kind, 0, cfg)
    assert (st["grid"] == 1) == one


@pytest.mark.parametrize("items", [511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 5000])
def test_tiles_of_a_small_worklist(irgl, items):
    """A source, `items` vertices, and 20 more behind each (shared)."""
    rng = np.random.default_rng(items)
    n = 1 + items + 10 * items
    u = np.concatenate([np.zeros(items, dtype=np.int64), np.repeat(1 + np.arange(items), 20)])
    v = np.concatenate([1 + np.arange(items), 1 + items + rng.integers(0, 10 * items, 20 * items)])
    g = gg.from_edges(n, u.tolist(), v.tolist(), (1 + np.arange(u.size) % 9).tolist())
    for cfg in ({"grid": 16, "block": 512}, {"grid": 64, "block": 256}, {"grid": 128, "block": 512},
                {"grid": 8, "block": 1024}):
        print(f"[case] {items} items {cfg}", flush=True)
        st = _check(irgl, g, BFS, 0, cfg)
        assert st["edges"] == u.size
