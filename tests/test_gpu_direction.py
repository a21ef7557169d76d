"""The default direction choice of BFS on symmetric graphs, on both sides of
the mean degree and of the skew where it changes: the levels are those of the
reference and of every explicit choice, single and batched, and top-down-only
graphs relax each reached vertex's row once."""
import numpy as np
import pytest

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu

BFS = 0


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


def _hub(n, d, hub):
    """A uniform graph whose vertex 0 also has `hub` neighbours."""
    rp, col, w = gg.uniform_random(n, d, seed=3, weight_seed=4).numpy()
    s = np.repeat(np.arange(n), np.diff(rp))
    keep = (s != 0) & (col != 0)
    u, v = s[keep].tolist(), col[keep].tolist()
    spokes = list(range(1, hub + 1))
    u, v = u + [0] * hub + spokes, v + spokes + [0] * hub
    g = gg.from_edges(n, u, v, [1] * len(u))
    g.symmetric = True
    return g


@pytest.mark.parametrize("make,top_down", [
    (lambda: gg.uniform_random(200000, 4.3, seed=3, weight_seed=4), True),
    (lambda: gg.uniform_random(200000, 4.7, seed=3, weight_seed=4), False),
    (lambda: gg.grid2d(301, weight_seed=4), True),
    (lambda: _hub(200000, 4.3, 60), True),
    (lambda: _hub(200000, 4.3, 80), False),
    (lambda: gg.rmat(14, 2, seed=3, weight_seed=4), False),
])
def test_default_direction(irgl, make, top_down):
    g = make()
    assert g.symmetric
    rp, col, _ = g.numpy()
    deg = np.diff(rp)
    for reorder in (False, True):
        hg = irgl.upload(g.to("cuda"), reorder=reorder)
        srcs = gg.pick_sources(g, 3, seed=5)
        refs = [oracle.bfs(rp, col, s)[0] for s in srcs]
        for src, ref in zip(srcs, refs):
            for cfg in (None, {"do_alpha": 4}, {"do_alpha": 10}, {"do_alpha": 0xFFFFFFFF}):
                print(f"[case] {g.name} src={src} reorder={reorder} {cfg}", flush=True)
                out, _, st = irgl.query(hg, BFS, src, with_parent=True, cfg=cfg)
                out = irgl.as_u32_numpy(out)
                np.testing.assert_array_equal(out, ref)
                if cfg is None:
                    whole = int(deg[out != 0xFFFFFFFF].sum())
                    assert (st["edges"] == whole) == top_down
        tasks = [irgl.Task(hg, BFS, s) for s in srcs]
        b = irgl.irgl_batch_submit(tasks)
        irgl.irgl_batch_wait(b)
        b.free()
        for task, ref in zip(tasks, refs):
            np.testing.assert_array_equal(irgl.as_u32_numpy(task.out), ref)


@pytest.mark.parametrize("path,width", [(3, 700), (900, 5000), (2100, 2100)])
def test_refreshes_of_the_visited_bitmap(irgl, path, width):
    """A path, then a fan of `width` vertices joined to one another, then a path."""
    a = list(range(path)) + [path] * width
    b = list(range(1, path + 1)) + [path + 1 + i for i in range(width)]
    rng = np.random.default_rng(path)
    a += [path + 1 + i for i in range(width)] * 2
    b += (path + 1 + rng.integers(0, width, 2 * width)).tolist()
    a += [path + width + i for i in range(path)]
    b += [path + 1 + width + i for i in range(path)]
    n = 2 * path + 1 + width
    g = gg.from_edges(n, a, b, [1] * len(a))
    rp, col, _ = g.numpy()
    ref, whole = oracle.bfs(rp, col, 0)[0], len(a)
    for symmetric in (False, True):
        if symmetric:
            g = gg.from_edges(n, a + b, b + a, [1] * (2 * len(a)))
            g.symmetric = True
            rp, col, _ = g.numpy()
            ref, whole = oracle.bfs(rp, col, 0)[0], 2 * len(a)
        hg = irgl.upload(g.to("cuda"))
        for t_bitmap in (0, 1, 64, width, 0xFFFFFFFF):
            for cfg in ({"grid": 4}, {"grid": 1, "block": 256}, {}):
                cfg = dict(cfg, t_bitmap=t_bitmap, do_alpha=0xFFFFFFFF)
                print(f"[case] {path} {width} symmetric={symmetric} {cfg}", flush=True)
                out, _, st = irgl.query(hg, BFS, 0, with_parent=True, cfg=cfg)
                np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
                assert st["edges"] == whole
