"""Batch and server launches up to the co-resident limits that explicit grids
rely on, per compute unit: 4 / 2 / 1 workgroups of 256 / 512 / 1024 threads in
a batch, 3 / 1 / 1 in a server; and solo runs inside teams at the sizes where
they begin and end.  Results are the oracle's, bit for bit."""
import time

import numpy as np
import pytest
import torch

import oracle
from paper_1607_05707_amd import graphgen as gg
from test_gpu_solo import GRAPHS

pytestmark = pytest.mark.gpu

BFS, SSSP = 0, 1
NAMES = ("path 1100", "brush 8 wide", "brush 513", "brush 1024", "brush 1025", "brush 2300", "brush 4097", "uniform 900",
         "directed 1500")


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


@pytest.fixture(scope="module")
def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


@pytest.fixture(scope="module")
def work(irgl):
    """(handle, kind, source, reference) of every task."""
    out = []
    graphs = [GRAPHS[k]() for k in NAMES] + [gg.rmat(12, 8, seed=3, weight_seed=4)]
    for g in graphs:
        rp, col, w = g.numpy()
        hg = irgl.upload(g.to("cuda"))
        for kind in (BFS, SSSP):
            ref = oracle.bfs(rp, col, 0)[0] if kind == BFS else oracle.dijkstra(rp, col, w, 0)[0]
            out.append((hg, kind, 0, ref))
    return out


CASES = [(256, 16, 4, 3), (512, 16, 2, 1), (1024, 16, 1, 1), (256, 1, 0, 0), (512, 3, 0, 0), (1024, 2, 0, 0)]


@pytest.mark.parametrize("block,team,in_batch,in_server", CASES)
def test_teams(irgl, cus, work, block, team, in_batch, in_server):
    cfg = {"block": block, "team": team, "grid": (in_batch * cus) or 12 * team}
    print(f"[case] batch {cfg}", flush=True)
    tasks = [irgl.Task(hg, kind, src) for hg, kind, src, _ in work]
    b = irgl.irgl_batch_submit(tasks, cfg=cfg)
    irgl.irgl_batch_wait(b)
    b.free()
    for t, (_, _, _, ref) in zip(tasks, work):
        np.testing.assert_array_equal(irgl.as_u32_numpy(t.out), ref)

    # gangs (tasks on the whole grid) between the teams' tasks
    cfg = {"block": block, "team": team, "grid": (in_server * cus) or 12 * team, "gang_edges": 5000}
    print(f"[case] server {cfg}", flush=True)
    server = irgl.irgl_batch_open([hg for hg, _, _, _ in work], cfg=cfg, ring_cap=64)
    tasks = [irgl.Task(hg, kind, src) for hg, kind, src, _ in work]
    tickets = [irgl.irgl_batch_enqueue(server, t) for t in tasks]
    assert None not in tickets
    t0 = time.time()
    left = set(tickets)
    while left:
        assert time.time() - t0 < 30.0, sorted(left)
        for k in sorted(left):
            st = irgl.irgl_batch_poll(server, k)
            if st is not None:
                assert st["status"] == 0
                left.discard(k)
    server.close()
    for t, (_, _, _, ref) in zip(tasks, work):
        np.testing.assert_array_equal(irgl.as_u32_numpy(t.out), ref)
