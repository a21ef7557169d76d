"""Solo runs (small invocations on one workgroup) and queries of one workgroup,
at the sizes where they begin and end.  Everything is exact against the
oracle."""
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


def _path(n):
    u = list(range(n - 1))
    return _symmetric(n, u, [x + 1 for x in u], [1 + (7 * x) % 50 for x in u])


def _brush(leaves, length):
    """A centre with `leaves` arms of `length` edges: worklists of `leaves`
    items, the first of them found through one row of `leaves` edges."""
    n = 1 + leaves * length
    u = [0 if j == 0 else 1 + i * length + j - 1 for i in range(leaves) for j in range(length)]
    v = [1 + i * length + j for i in range(leaves) for j in range(length)]
    return _symmetric(n, u, v, [1 + (5 * i) % 90 for i in range(len(u))])


GRAPHS = {
    "path 2": lambda: _path(2),
    "path 1100": lambda: _path(1100),             # more steps than one solo run takes
    "brush 3": lambda: _brush(3, 40),
    "brush 8 wide": lambda: _brush(9, 30),        # a row longer than one thread walks
    "brush 511": lambda: _brush(511, 3),
    "brush 513": lambda: _brush(513, 3),
    "brush 1024": lambda: _brush(1024, 3),
    "brush 1025": lambda: _brush(1025, 3),        # past the items of a run
    "brush 2300": lambda: _brush(2300, 2),        # past the LDS worklist of 256 threads
    "brush 4097": lambda: _brush(4097, 2),        # past the edges of a run
    "grid 40x57": lambda: gg.grid2d(40, 57, weight_seed=3, wmax=100),
    "road 96": lambda: gg.config_road(width=96),
    "uniform 900": lambda: gg.uniform_random(900, 18.0, seed=4, weight_seed=5),
    "rmat 11": lambda: gg.rmat(11, 6, seed=6, weight_seed=7),
    "directed 1500": lambda: gg.random_directed(1500, 5200, seed=8, weight_seed=9),
}


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


@pytest.mark.parametrize("name", list(GRAPHS))
def test_small_worklists(irgl, name):
    cpu = GRAPHS[name]()
    g = cpu.to("cuda")
    src = gg.pick_sources(cpu, 1, seed=1)[0] if name.startswith(("uniform", "rmat", "directed")) else 0
    for reorder in (False, True):
        hg = irgl.upload(g, reorder=reorder)
        for kind in (BFS, SSSP):
            # default (one workgroup where the graph is small), a few
            # workgroups, and a full grid of each size
            for cfg in (None, {"grid": 8}, {"block": 256, "grid": 24}, {"block": 512, "grid": 256},
                        {"block": 1024, "grid": 256}):
                st = _check(irgl, cpu, hg, kind, src, cfg)
                if cfg and "grid" in cfg:
                    assert st["grid"] == cfg["grid"]
            if kind == SSSP and name in ("grid 40x57", "road 96", "directed 1500"):
                for delta in (1, 40, 3000):  # far lists of every size, from one entry per bucket on
                    _check(irgl, cpu, hg, kind, src, {"delta": delta, "grid": 64})
                    _check(irgl, cpu, hg, kind, src, {"delta": delta})


def test_limits_inside_a_solo_run(irgl):
    """The iteration limit and the worklist capacity are kept by solo runs."""
    cpu = _path(600)
    hg = irgl.upload(cpu.to("cuda"))
    for cfg in ({"max_iter": 77}, {"max_iter": 77, "grid": 16}):
        out, _, st = irgl.query(hg, BFS, 0, cfg=cfg, check=False)
        assert st["status"] == irgl.IRGL_ERR_ITERATION_LIMIT and st["iterations"] == 77
        lv = irgl.as_u32_numpy(out)
        assert int((lv != oracle.INF).sum()) == 78
    brush = _brush(40, 3)
    hb = irgl.upload(brush.to("cuda"))
    for cfg in ({"wl_capacity": 39}, {"wl_capacity": 39, "grid": 16}):
        _, _, st = irgl.query(hb, BFS, 0, cfg=cfg, check=False)
        assert st["status"] == irgl.IRGL_ERR_OVERFLOW
    _check(irgl, brush, hb, BFS, 0, {"wl_capacity": 40})
