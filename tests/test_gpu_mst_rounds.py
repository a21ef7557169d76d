"""Minimum spanning forest: the sizes where a round's shortcuts begin and end
(rows around a lane's four entries and the workgroup's row, hook chains longer
than one pass follows, a dominant component that is skipped, lightest edges
kept from the round before), bit for bit against Kruskal."""
import numpy as np
import pytest

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


def _graph(n, u, v, w):
    return gg.from_edges(n, list(u) + list(v), list(v) + list(u), list(w) + list(w))


def _rising_path(n):
    """Every vertex's lightest edge leads to its left: one chain of n hooks."""
    return _graph(n, range(n - 1), range(1, n), range(1, n))


def _rows(k):
    """Circulant graph of even degree k on 640 vertices: every row has k entries."""
    n, half = 640, k // 2
    u = [i for i in range(n) for _ in range(half)]
    v = [(i + d) % n for i in range(n) for d in range(1, half + 1)]
    return _graph(n, u, v, [1 + (i * 37) % 101 for i in range(len(u))])


def _hub(leaves, islands):
    """A hub joined to its leaves (half of them in pairs), and `islands` edges
    and single vertices beside it."""
    n = 1 + leaves + 3 * islands
    u, v, w = [0] * leaves, list(range(1, leaves + 1)), [5 + i % 9 for i in range(leaves)]
    for i in range(1, leaves // 2, 2):
        u.append(i), v.append(i + 1), w.append(1 + i % 4)
    for k in range(islands):
        a = 1 + leaves + 3 * k
        u.append(a), v.append(a + 1), w.append(7)
    return _graph(n, u, v, w)


def _two_halves(n):
    """Two uniform graphs of n vertices, joined by three heavy edges: each half
    grows on its own before they meet."""
    a = gg.uniform_random(n, 6.0, seed=n, weight_seed=n + 1, wmax=50)
    rp, col, w = a.numpy()
    s = np.repeat(np.arange(n), np.diff(rp))
    keep = s < col
    u, v, x = s[keep].tolist(), col[keep].tolist(), w[keep].tolist()
    u2, v2 = [i + n for i in u], [i + n for i in v]
    return _graph(2 * n, u + u2 + [0, 1, 2], v + v2 + [n, n + 1, n + 2], x + x + [900, 901, 902])


GRAPHS = {f"path {n}": (lambda n=n: _rising_path(n)) for n in (2, 33, 34, 35, 1200, 40000)}
GRAPHS.update({f"rows of {k}": (lambda k=k: _rows(k)) for k in (2, 4, 6, 8, 10)})
GRAPHS.update({f"hub {k}": (lambda k=k: _hub(k, 70)) for k in (90, 4095, 4096, 4097, 16390)})
GRAPHS["two halves"] = lambda: _two_halves(3000)
GRAPHS["rmat 13"] = lambda: gg.rmat(13, 16, seed=5, weight_seed=6)


@pytest.mark.parametrize("name", list(GRAPHS))
def test_rounds(irgl, name):
    g = GRAPHS[name]()
    ref_w, ref_f, ref_c, ref_ne = oracle.kruskal(*g.numpy())
    hg = irgl.upload(g.to("cuda"))
    for lock in (0, 1, 2):
        for cfg in ({"lock": lock}, {"lock": lock, "block": 256, "grid": 3}, {"lock": lock, "block": 1024}):
            if lock and name == "hub 16390":
                continue  # thousands of lock holders on one component, one after another
            print(f"[case] mst {name} {cfg}", flush=True)
            weight, comp, marks, st = irgl.mst(hg, cfg=cfg)
            assert weight == ref_w and st["frontier_edges"] == ref_ne
            np.testing.assert_array_equal(marks.cpu().numpy(), ref_f)
            np.testing.assert_array_equal(comp.cpu().numpy(), ref_c)
