"""Multi-source searches on relabeled graphs, whose results pass through
cells in label space: root counts at the edges of the cells' stride and of a
batch, searches deeper than a byte holds (254, 255 and 300 levels), bounded
depths, no parents, vertex counts around the transposing tile.  Whole
numbers: every row equals a search from its root alone (sampled against the
oracle)."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _path(n):
    return gg.csr_from_edges(n, [(i, i + 1) for i in range(n - 1)])


GRAPHS = {
    "kron13": lambda: gg.kronecker(13, 16, seed=2),
    "n63": lambda: gg.random_graph(63, 0.1, 3),
    "n65": lambda: gg.random_graph(65, 0.05, 4),
    "path255": lambda: _path(255),
    "path256": lambda: _path(256),
    "path301": lambda: _path(301),
}


@pytest.mark.parametrize("enc", [dict(ids="local", offsets="ef"), dict(layout="plain")], ids=["local-ef", "plain"])
@pytest.mark.parametrize("relabel", ["degree", "greedy"])
@pytest.mark.parametrize("name", GRAPHS)
def test_cells(name, relabel, enc):
    g = GRAPHS[name]()
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, relabel=relabel, **enc)
    rng = np.random.default_rng(5)
    for count in (16, 17, 64, 80):
        roots = [0, g.n - 1] + [int(x) for x in rng.integers(0, g.n, count - 2)]
        for depth, parent in ((-1, True), (2, True), (-1, False)):
            d, p = lg.bfs(h, roots, max_depth=depth, parent=parent)
            for i in list(range(4)) + [15, count - 1]:
                d1, p1 = lg.bfs(h, [roots[i]], max_depth=depth, parent=parent)
                assert torch.equal(d[i], d1[0]), (count, depth, i)
                assert not parent or torch.equal(p[i], p1[0]), (count, depth, i)
            d0, _ = orc.bfs(off, col, roots[1], max_depth=depth)
            assert np.array_equal(d[1].cpu().numpy(), d0)
    h.free()
