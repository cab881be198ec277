"""Top-down levels large enough that their claims are binned by vertex
(from 2^20 vertices and 2^20 edges): a vertex count that ends inside a bin
and a bitmap word, and neighbors crowded into two of the bins, so that their
room runs out.  Whole numbers: equal to the oracle's."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

N = (1 << 20) + 77
EDGES = 55 * N


def _graph(crowded):
    gen = torch.Generator(device="cuda").manual_seed(11)
    src = torch.randint(0, N, (EDGES,), generator=gen, device="cuda")
    dst = torch.randint(0, N, (EDGES,), generator=gen, device="cuda")
    if crowded:
        dst[: EDGES // 10] %= N // 32
    return gg.canonical_csr(N, src, dst)


def _root(g, off, col):
    """A root with a level of 2^20 edges or more that is searched top-down (at
    most a sixtieth of the entries not yet seen), and its oracle results."""
    deg = np.diff(off.astype(np.int64))
    for root in range(N - 1, 0, -9973):
        depth, parent = orc.bfs(off, col, root)
        left = g.m
        for level in range(int(depth.max())):
            edges = int(deg[depth == level].sum())
            if edges > left // 60:
                break
            if edges >= 1 << 20:
                return root, depth, parent
            left -= edges
    raise AssertionError("no root with such a level")


@pytest.mark.parametrize("crowded", [False, True])
def test_binned_levels(crowded):
    g = _graph(crowded)
    off, col = g.numpy()
    root, d0, p0 = _root(g, off, col)
    for enc in (dict(ids="local", offsets="ef"), dict(layout="plain"), dict(relabel="degree")):
        h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **enc)
        d, p = lg.bfs(h, [root])
        assert np.array_equal(d[0].cpu().numpy(), d0), enc
        if "relabel" not in enc:  # (relabeled: the smallest label's parent)
            assert np.array_equal(p[0].cpu().numpy(), p0), enc
        d1, _ = lg.bfs(h, [root], parent=False)
        assert torch.equal(d1, d), enc
        h.free()
