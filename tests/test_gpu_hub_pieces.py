"""Few grid-tier chunks cut into pieces over the workgroups, at the sizes where
the pieces change.  Everything is exact against the oracle."""
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


def _symmetric(n, u, v, w):
    g = gg.from_edges(n, u + v, v + u, w + w)
    g.symmetric = True
    return g


def _brush(leaves, length):
    """A centre with `leaves` arms of `length` edges: worklists of `leaves`
    items, the first of them found through one row of `leaves` edges."""
    n = 1 + leaves * length
    u = [0 if j == 0 else 1 + i * length + j - 1 for i in range(leaves) for j in range(length)]
    v = [1 + i * length + j for i in range(leaves) for j in range(length)]
    return _symmetric(n, u, v, [1 + (5 * i) % 90 for i in range(len(u))])


def _check(irgl, g, hg, kind, src, cfg):
    print(f"[case] kind={kind} src={src} cfg={cfg}", flush=True)
    rp, col, w = g.numpy()
    out, par, st = irgl.query(hg, kind, src, with_parent=True, cfg=cfg)
    ref = oracle.bfs(rp, col, src)[0] if kind == BFS else oracle.dijkstra(rp, col, w, src)[0]
    np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
    oracle.validate(rp, col, src, ref, par.cpu().numpy(), None if kind == BFS else w)
    if kind == BFS:
        assert st["iterations"] == int(ref[ref != oracle.INF].max()) + 1
        assert st["items"] == int((ref != oracle.INF).sum())
        assert st["frontier_edges"] == oracle.edges_scanned(rp, ref)
    return st


@pytest.mark.parametrize("leaves", [255, 256, 257, 4095, 4097, 9000, 70000])
def test_few_grid_tier_chunks(irgl, leaves):
    """One row of `leaves` edges in the grid tier, cut into pieces over the
    workgroups; the rows that lead back are short."""
    cpu = _brush(leaves, 1)
    hg = irgl.upload(cpu.to("cuda"))
    for kind in (BFS, SSSP):
        for src in (0, leaves):
            for cfg in ({"t_grid": 64, "t_block": 64, "grid": 96}, {"grid": 7}, {"block": 256, "grid": 256},
                        {"block": 1024, "grid": 256}):
                _check(irgl, cpu, hg, kind, src, cfg)
