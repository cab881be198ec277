"""SSSP where a collecting workgroup takes more than one tile of the bitmap
(above 2,048 tiles of 64 words: 2^23 vertices), so that places run on from
tile to tile, with marks all over the bitmap, in its first words only (degree
relabeling) and, after the search's end, none.  Distances are whole numbers:
equal to the oracle's Dijkstra."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", params=[(1 << 23) - 63, (1 << 23) + 1, (1 << 23) + 5000, 3 << 22])
def graph(request):
    """A hub tied to 100,000 vertices all over the labels, edges among them,
    and a chain of labels through the whole range."""
    n = request.param
    rng = np.random.default_rng(n)
    some = np.unique(rng.integers(1, n, 100000))
    chain = np.sort(rng.choice(some, 200, replace=False))
    chain[-1] = n - 1
    src = np.concatenate([np.zeros(len(some) // 2, np.int64), rng.choice(some, 150000), chain[:-1]])
    dst = np.concatenate([some[: len(some) // 2], rng.choice(some, 150000), chain[1:]])
    g = gg.canonical_csr(n, torch.from_numpy(src), torch.from_numpy(dst))
    w = gg.edge_weights(g, 255, 5)
    off, col = g.numpy()
    want = orc.sssp(off.astype(np.uint64), col.view(np.uint32), w.numpy().astype(np.uint32), n - 1)
    return g, w, want


@pytest.mark.parametrize("enc", [dict(ids="local", offsets="ef"), dict(ids="global", relabel=True), dict(layout="plain")],
                         ids=["local-ef", "global-dm", "plain"])
def test_tiles(graph, enc):
    g, w, want = graph
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, weights=w.cuda(), **enc)
    for delta in (0, 40):
        assert np.array_equal(lg.sssp(h, g.n - 1, delta).cpu().numpy(), want), delta
    h.free()
