"""Calls of up to 15 roots on small graphs, which run in one launch: graphs on
both sides of the rule's vertex and entry counts, hub lists beside short
ones, many levels, edgeless graphs, bounded depths, no parents, repeated
roots.  Whole numbers: depths equal to the oracle's, parents to it or (where
relabeled) to a top-down search's."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

ENCODINGS = {
    "global": dict(),
    "plain-dm": dict(layout="plain", relabel="degree"),
    "local-ef-dm": dict(ids="local", offsets="ef", relabel="degree"),
    "gap-greedy": dict(ids="local-gap", offsets="ef", relabel="greedy"),
    "varint-diff-dm": dict(ids="varint-diff", relabel="degree"),
}


def _hubs(n, hubs):
    return gg.csr_from_edges(n, [(h, v) for h in range(hubs) for v in range(hubs, n)])


GRAPHS = {
    "one": lambda: gg.csr_from_edges(1, []),
    "edgeless": lambda: gg.csr_from_edges(130, []),
    "path": lambda: gg.csr_from_edges(400, [(i, i + 1) for i in range(399)]),
    "hubs": lambda: _hubs(1500, 9),
    "kron10": lambda: gg.kronecker(10, 16, seed=3),
    "er-16384": lambda: gg.random_graph(1 << 14, 0.0005, 4),
    "er-16385": lambda: gg.random_graph((1 << 14) + 1, 0.0005, 4),
    "entries-2^18": lambda: _hubs((1 << 14), 8),
    "kron13": lambda: gg.kronecker(13, 16, seed=5),
    "kron14": lambda: gg.kronecker(14, 16, seed=5),
}


@pytest.mark.parametrize("enc", ENCODINGS)
@pytest.mark.parametrize("name", GRAPHS)
def test_small(name, enc):
    g = GRAPHS[name]()
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **ENCODINGS[enc])
    rng = np.random.default_rng(6)
    for count in (1, 2, 15):
        roots = [int(x) for x in rng.integers(0, g.n, count)]
        if count > 1:
            roots[-1] = roots[0]
        for depth, parent in ((-1, True), (0, True), (2, False), (2, True)):
            d, p = lg.bfs(h, roots, max_depth=depth, parent=parent)
            for i in {0, count // 2, count - 1}:
                d0, p0 = orc.bfs(off, col, roots[i], max_depth=depth)
                assert np.array_equal(d[i].cpu().numpy(), d0), (count, depth, i)
                if parent and "relabel" not in ENCODINGS[enc]:
                    assert np.array_equal(p[i].cpu().numpy(), p0), (count, depth, i)
                elif parent:
                    _, p1 = lg.bfs(h, [roots[i]], max_depth=depth, mode="td")
                    assert torch.equal(p[i], p1[0]), (count, depth, i)
