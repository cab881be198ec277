"""Timing kernels while a plan is created, which captures its launch in a
graph: the capture is not timed, and later calls and timings are sound."""

import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def test_calls_after_a_timed_plan():
    g = gg.kronecker(10, 8, seed=1)
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n)
    root = gg.pick_roots(g, 1, seed=1)[0]
    lg.prof_reset()
    lg.prof_enable(True)
    plan = lg.BatchPlan([h], [(0, root)], autotune=False)
    assert lg.prof_query("batch_reset_kernel")[0] == 1  # the one run of the creation
    d, p = lg.bfs(h, [root], mode="td")
    plan.run()
    torch.cuda.synchronize()
    assert lg.prof_query("bfs_init_kernel")[0] == 1
    lg.prof_enable(False)
    assert torch.equal(plan.depth(0), d[0]) and torch.equal(plan.parent(0), p[0])
    plan.free()
    h.free()
    lg.prof_reset()
