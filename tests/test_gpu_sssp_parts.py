"""SSSP at vertex counts where the collecting workgroups' ranges change: one
range, the last range short, more words than ranges times a wave (2^18
vertices and one more), marks in the first words only (degree relabeling),
chains longer than the steps queued between two looks.  Distances are whole
numbers: equal to the oracle's Dijkstra."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _uniform(n, m, seed):
    rng = np.random.default_rng(seed)
    return gg.canonical_csr(n, torch.from_numpy(rng.integers(0, n, m)), torch.from_numpy(rng.integers(0, n, m)))


GRAPHS = {
    "n255": lambda: _uniform(255, 800, 1),
    "n257": lambda: _uniform(257, 800, 2),
    "n16385": lambda: _uniform(16385, 60000, 3),
    "n262144": lambda: _uniform(262144, 600000, 4),
    "n262209": lambda: _uniform(262209, 600000, 5),
    "n1100000": lambda: _uniform(1100000, 1500000, 6),
    "kron16": lambda: gg.kronecker(16, 8, seed=7),
    "path90": lambda: gg.csr_from_edges(90, [(i, i + 1) for i in range(89)]),
}


@pytest.mark.parametrize("enc", [dict(ids="local", offsets="ef"), dict(ids="global", relabel=True), dict(layout="plain")],
                         ids=["local-ef", "global-dm", "plain"])
@pytest.mark.parametrize("name", GRAPHS)
def test_parts(name, enc):
    g = GRAPHS[name]()
    w = gg.edge_weights(g, 255, 9)
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, weights=w.cuda(), **enc)
    for root in (0, g.n - 1):
        want = orc.sssp(off.astype(np.uint64), col.view(np.uint32), w.numpy().astype(np.uint32), root)
        for delta in (0, 50):
            assert np.array_equal(lg.sssp(h, root, delta).cpu().numpy(), want), (root, delta)
    h.free()
