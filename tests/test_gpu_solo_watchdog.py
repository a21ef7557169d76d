"""Solo runs under a small watchdog: the other workgroups wait at one barrier
while a run lasts, so it has to end well before the bound.  (Before it did,
512 invocations of a thousand items each took longer than the bound.)"""
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


def _brush(leaves, length):
    """A centre with `leaves` arms of `length` edges: `length` worklists of
    `leaves` items one after another."""
    e = np.arange(leaves * length)
    u, v = np.where(e % length == 0, 0, e), 1 + e
    w = 1 + (5 * e) % 9
    g = gg.from_edges(1 + leaves * length, np.concatenate([u, v]).tolist(), np.concatenate([v, u]).tolist(),
                      np.concatenate([w, w]).tolist())
    g.symmetric = True
    return g


@pytest.mark.parametrize("leaves,length", [(1, 9000), (1000, 600), (480, 900)])
def test_a_solo_run_keeps_a_small_watchdog(irgl, leaves, length):
    g = _brush(leaves, length)
    assert g.n > 8192  # more than one workgroup by default
    rp, col, w = g.numpy()
    hg = irgl.upload(g.to("cuda"))
    for kind, ref in ((BFS, oracle.bfs(rp, col, 0)[0]), (SSSP, oracle.dijkstra(rp, col, w, 0)[0])):
        for cfg in ({}, {"grid": 8}, {"grid": 200, "block": 256}):
            cfg = dict(cfg, watchdog_ms=1)
            print(f"[case] brush {leaves} x {length} kind={kind} {cfg}", flush=True)
            out, _, st = irgl.query(hg, kind, 0, with_parent=False, cfg=cfg)
            assert st["status"] == 0
            np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
