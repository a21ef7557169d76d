"""Batch tasks are taken longest first.  One team runs them one after another
into one output, which holds the last task's result."""
import numpy as np
import pytest
import torch

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu

BFS = 0


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


# (vertices, mean degree) of the longer and of the shorter BFS.  Below a mean
# degree of 4.5 a BFS stays top-down and scans every entry (577 us for 260,000
# vertices); above, it goes bottom-up and scans few (254 us for 100,000).
@pytest.mark.parametrize("longer,shorter", [((260000, 4.2), (350000, 12.0)), ((350000, 12.0), (100000, 4.2)),
                                            ((200000, 6.0), (100000, 12.0))])
def test_the_longer_task_runs_first(irgl, longer, shorter):
    graphs = [gg.uniform_random(n, d, seed=3, weight_seed=4) for n, d in (longer, shorter)]
    handles = [irgl.upload(g.to("cuda")) for g in graphs]
    srcs = [gg.pick_sources(g, 1, seed=5)[0] for g in graphs]
    out = torch.empty(max(g.n for g in graphs), dtype=torch.int32, device="cuda")
    last = graphs[1]
    ref = oracle.bfs(*last.numpy()[:2], srcs[1])[0]
    for order in ((0, 1), (1, 0)):
        print(f"[case] {longer} before {shorter}, submitted {order}", flush=True)
        tasks = [irgl.Task(handles[k], BFS, srcs[k], out=out[:graphs[k].n]) for k in order]
        b = irgl.irgl_batch_submit(tasks, cfg={"block": 512, "team": 16, "grid": 16})
        irgl.irgl_batch_wait(b)
        b.free()
        np.testing.assert_array_equal(irgl.as_u32_numpy(out[:last.n]), ref)
