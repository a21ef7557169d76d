"""SSSP far lists handed between a solo run and the team: a star whose centre
lists every leaf at once and leaves the worklist empty, with far lists on both
sides of what a solo run transfers (2048 entries) and of the edges it scans
(4096).  The trace says which invocations one workgroup ran alone: the largest
and the summed busy ticks (words 7 and 8) are then the same."""
import numpy as np
import pytest
import torch

import oracle
from paper_1607_05707_amd import graphgen as gg

pytestmark = pytest.mark.gpu

SSSP, WORDS = 1, 12


@pytest.fixture(scope="module")
def irgl():
    from paper_1607_05707_amd import irgl as m
    return m


def _star(leaves):
    """A centre, its leaves at weights from 10 on, and a vertex beyond every fifth leaf."""
    i = np.arange(leaves)
    far = i[::5]
    u = np.concatenate([np.zeros(leaves, dtype=np.int64), 1 + far])
    v = np.concatenate([1 + i, 1 + leaves + np.arange(far.size)])
    w = np.concatenate([10 + i * 13 % 40, 1 + far % 9])
    g = gg.from_edges(1 + leaves + far.size, np.concatenate([u, v]).tolist(), np.concatenate([v, u]).tolist(),
                      np.concatenate([w, w]).tolist())
    g.symmetric = True
    return g


@pytest.mark.parametrize("leaves", [1, 2047, 2048, 2049, 4000, 4096, 4097])
def test_far_lists_between_solo_runs_and_the_team(irgl, leaves):
    g = _star(leaves)
    rp, col, w = g.numpy()
    ref = oracle.dijkstra(rp, col, w, 0)[0]
    hg = irgl.upload(g.to("cuda"))
    for delta in (1, 5, 45):
        for block in (256, 512, 1024):
            tr = torch.zeros(WORDS * 1024 + 1, dtype=torch.int64, device="cuda")
            cfg = {"delta": delta, "grid": 64, "block": block, "trace": tr, "trace_len": tr.numel()}
            print(f"[case] star {leaves} delta={delta} block={block}", flush=True)
            out, par, st = irgl.query(hg, SSSP, 0, with_parent=True, cfg=cfg)
            np.testing.assert_array_equal(irgl.as_u32_numpy(out), ref)
            oracle.validate(rp, col, 0, ref, par.cpu().numpy(), w)
            it = st["iterations"]
            assert 0 < it < 1024
            t = tr.cpu().numpy()[:WORDS * it].reshape(it, WORDS)
            ran = t[:, 8] > 0
            alone = ran & (t[:, 7] == t[:, 8])
            assert bool(alone[0]) == (leaves <= 4096)  # the centre's row
            assert t[0][1] == 1 and t[0][2] == leaves
            if delta == 1 and leaves > 1:
                assert alone[1:].any()  # buckets of a few leaves each
