"""PageRank with fixed places (tiles of source blocks and destination bins):
vertex counts at the edges of blocks, bins and their shape changes, hub bins
shared by several workgroups, empty blocks, every encoding, and iteration
counts on both sides of the line between it and the pull.

Tolerance: the sums are exact, so an iteration rounds a contribution twice
(score and quotient) and the score once, each by 2^-24 of its value, and the
base term once: after t iterations a score is off by at most (4 t + 2) 2^-24
of itself, plus the fixed-point unit 2^-61 per entry and iteration.  The pull
(few iterations on decoded encodings) adds in FP32 and is held to L1 1e-5."""

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


def _hub(n, seed):
    """One vertex tied to two thirds of the others, the last third without edges."""
    k = 2 * n // 3
    leaves = torch.arange(1, k)
    rng = np.random.default_rng(seed)
    a, b = torch.from_numpy(rng.integers(0, k, k)), torch.from_numpy(rng.integers(0, k, k))
    return gg.canonical_csr(n, torch.cat([torch.zeros(k - 1, dtype=torch.int64), a]), torch.cat([leaves, b]))


GRAPHS = {
    "n1024": lambda: _uniform(1024, 3000, 1),
    "n1025-hub": lambda: _hub(1025, 2),
    "n8191": lambda: _uniform(8191, 40000, 3),
    "n8193": lambda: _uniform(8193, 40000, 4),
    "n65536-kron": lambda: gg.kronecker(16, 16, seed=5),
    "n65537-hub": lambda: _hub(65537, 6),
    "n524289-hub": lambda: _hub(524289, 7),
    "n1048575": lambda: _uniform(1048575, 1 << 20, 8),
    "n1048577": lambda: _uniform(1048577, 1 << 20, 9),
    "n2097153-sparse": lambda: _uniform(2097153, 50000, 10),
    "n4096-none": lambda: gg.csr_from_edges(4096, []),
    "n1500-dense": lambda: gg.random_graph(1500, 0.8, 11),
}
OPTS = [dict(ids="global", offsets="packed"), dict(layout="plain"), dict(ids="local", offsets="ef", relabel=True),
        dict(ids="local-gap", offsets="packed"), dict(ids="varint-diff", offsets="ef", relabel="greedy")]


@pytest.fixture(scope="module", params=list(GRAPHS))
def graph(request):
    g = GRAPHS[request.param]()
    off, col = g.numpy()
    off, col = off.astype(np.uint64), col.view(np.uint32)
    want = {t: orc.pagerank_par(off, col, 0.85, t) for t in (1, 12)}
    return request.param, g, want


@pytest.mark.parametrize("opts", OPTS, ids=lambda o: "-".join(map(str, o.values())))
def test_tiles(graph, opts):
    name, g, want = graph
    dg = g.to("cuda")
    h = lg.encode(dg.row_offsets, dg.col, g.n, **opts)
    for t in (1, 12):
        pr = lg.pagerank(h, 0.85, t)
        assert torch.equal(pr, lg.pagerank(h, 0.85, t))
        got = pr.cpu().numpy().astype(np.float64)
        ref = np.asarray(want[t], dtype=np.float64)
        if t >= 10 or opts.get("ids", "global") == "global":
            off = np.abs(got - ref)
            deg = np.diff(g.numpy()[0])
            assert (off <= (4 * t + 2) * 2.0 ** -24 * ref + t * (deg + 1) * 2.0 ** -61).all(), (name, t, off.max())
        assert np.abs(got - ref).sum() <= 1e-5
    h.free()
