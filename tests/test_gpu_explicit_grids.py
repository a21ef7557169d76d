"""Explicit grids up to the co-resident limits that callers rely on, per
compute unit: 4 / 2 / 1 workgroups of 256 / 512 / 1024 threads for BFS, 5 / 2
/ 1 for SSSP and the spanning forest, 6 / 12 of 256 / 128 for refinement.
(With more registers per thread the larger ones were refused.)"""
import numpy as np
import pytest
import torch

import oracle
from oracle import mesh as om
from paper_1607_05707_amd import graphgen as gg
from paper_1607_05707_amd import meshgen

pytestmark = pytest.mark.gpu

BFS, SSSP = 0, 1


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


@pytest.fixture(scope="module")
def cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


QUERY_GRAPHS = {  # on one workgroup by default, solo runs, skewed (no solo runs), directed
    "grid 64": lambda: gg.config_grid64(),
    "uniform": lambda: gg.uniform_random(20000, 6.0, seed=3, weight_seed=4),
    "rmat 15": lambda: gg.rmat(15, 8, seed=5, weight_seed=6),
    "directed": lambda: gg.random_directed(12000, 70000, seed=7, weight_seed=8),
}


@pytest.mark.parametrize("name", list(QUERY_GRAPHS))
def test_query_grids(irgl, cus, name):
    g = QUERY_GRAPHS[name]()
    rp, col, w = g.numpy()
    src = gg.pick_sources(g, 1, seed=2)[0]
    hg = irgl.upload(g.to("cuda"))
    for kind, per_cu in ((BFS, {256: 4, 512: 2, 1024: 1}), (SSSP, {256: 5, 512: 2, 1024: 1})):
        ref = oracle.bfs(rp, col, src)[0] if kind == BFS else oracle.dijkstra(rp, col, w, src)[0]
        for block, k in per_cu.items():
            cfg = {"block": block, "grid": k * cus}
            print(f"[case] {name} kind={kind} {cfg}", flush=True)
            out, _, st = irgl.query(hg, kind, src, with_parent=True, cfg=cfg)
            assert st["grid"] == k * cus and st["block"] == block
            np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)


def test_forest_grids(irgl, cus):
    g = gg.rmat(12, 6, seed=9, weight_seed=10)
    rp, col, w = g.numpy()
    ref, _, comp, _ = oracle.kruskal(rp, col, w)
    hg = irgl.upload(g.to("cuda"))
    for block, k in ((256, 5), (512, 2), (1024, 1)):
        print(f"[case] forest {block} x {k * cus}", flush=True)
        weight, c, _, st = irgl.mst(hg, cfg={"block": block, "grid": k * cus})
        assert weight == ref and st["grid"] == k * cus
        np.testing.assert_array_equal(c.cpu().numpy(), comp)


@pytest.mark.parametrize("block,k", [(256, 6), (128, 12), (64, 24)])
def test_refinement_grids(irgl, cus, block, k):
    m = meshgen.random_square(400, 5)
    dm = irgl.DeviceMesh.from_host(m, torch.device("cuda:0"))
    print(f"[case] refinement {block} x {k * cus}", flush=True)
    st = irgl.dmr(dm, {"block": block, "grid": k * cus})
    assert st["final_bad"] == 0
    om.check_mesh(dm.pts[:dm.npts].cpu().numpy(), dm.tri[:dm.ntri].cpu().numpy(), dm.nbr[:dm.ntri].cpu().numpy(),
                  input_pts=m.input_pts, min_angle=30.0)


def test_grids_left_at_zero(irgl, cus):
    """The workgroups of launches whose grid is left at 0 do not follow the limits."""
    g = gg.uniform_random(60000, 6.0, seed=3, weight_seed=4)
    rp, col, _ = g.numpy()
    src = gg.pick_sources(g, 1, seed=2)[0]
    ref = oracle.bfs(rp, col, src)[0]
    hg = irgl.upload(g.to("cuda"))
    for block in (256, 512, 1024):
        _, _, st = irgl.query(hg, BFS, src, cfg={"block": block})
        assert st["grid"] == cus * max(1, 512 // block)
    weight, _, _, st = irgl.mst(hg, cfg={"block": 256})
    assert weight == oracle.kruskal(*g.numpy())[0] and st["grid"] <= cus * 4
    level = torch.empty(g.n, dtype=torch.int32, device="cuda")
    for block in (64, 128, 256, 512, 1024):
        print(f"[case] pipe {block}", flush=True)
        stats = irgl.stats_tensor(torch.device("cuda:0"))
        irgl.irgl_pipe_run(hg, irgl.pipe_bfs_program(), src=src, level=level, block=block, stats=stats)
        st = irgl.read_stats(stats)
        assert st["status"] == 0 and st["grid"] == cus * max(1, 512 // block)
        np.testing.assert_array_equal(irgl.as_u32_numpy(level), ref)
