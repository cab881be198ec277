"""The two kernels of batched BFS under their own names in the profile: plans
up to 349,504 vertices (whose bitmaps fill 128 KB) and from 349,505."""

import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,name,other", [(349504, "bfs_batch_kernel", "bfs_batch_large_kernel"),
                                          (349505, "bfs_batch_large_kernel", "bfs_batch_kernel")])
def test_names(n, name, other):
    g = gg.csr_from_edges(n, [(0, n - 1), (n - 1, 5)])
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n)
    lg.prof_reset()
    lg.prof_enable(True)
    plan = lg.BatchPlan([h], [(0, 0), (0, 5)], autotune=False)
    lg.prof_enable(False)
    assert lg.prof_query(name)[0] >= 1 and lg.prof_query(other)[0] == 0
    plan.run()
    torch.cuda.synchronize()
    assert int(plan.depth(0)[5]) == 2 and int(plan.depth(1)[0]) == 2
    plan.free()
    h.free()
    lg.prof_reset()
