"""Decodes whose output is cut into wave pieces: list lengths and request
orders that put piece edges inside long lists, at list ends and in runs of
empty lists.  The lists are whole numbers: the results equal the input."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _ragged(n, hub, seed):
    """A hub, lists of 1-3 entries, and long runs of vertices without edges."""
    rng = np.random.default_rng(seed)
    edges = [(0, int(v)) for v in rng.choice(np.arange(1, n), hub, replace=False)]
    lo, hi = n // 2, n // 2 + n // 8
    edges += [(int(a), int(b)) for a, b in zip(rng.integers(lo, hi, n // 8), rng.integers(lo, hi, n // 8)) if a != b]
    return gg.csr_from_edges(n, edges)


GRAPHS = {
    "hub-9000": lambda: _ragged(40000, 9000, 1),
    "hub-255": lambda: _ragged(700, 255, 2),
    "hub-256": lambda: _ragged(700, 256, 3),
    "kron15": lambda: gg.kronecker(15, 16, seed=4),
}
OPTS = [dict(ids="global", offsets="packed"), dict(ids="local", offsets="ef"), dict(layout="plain"),
        dict(ids="global", offsets="interleaved-bv"), dict(ids="local", offsets="ef", relabel=True)]


@pytest.mark.parametrize("opts", OPTS, ids=lambda o: "-".join(map(str, o.values())))
@pytest.mark.parametrize("name", GRAPHS)
def test_pieces(name, opts):
    g = GRAPHS[name]()
    off, col = g.numpy()
    dg = g.to("cuda")
    h = lg.encode(dg.row_offsets, dg.col, g.n, **opts)
    rng = np.random.default_rng(9)
    requests = {
        "all": np.arange(g.n),
        "shuffled": rng.permutation(g.n),
        "repeated hub": np.repeat(int(np.argmax(np.diff(off))), 70),
        "empty before and after": np.concatenate([np.full(200, g.n - 1), [0, 0, 1], np.full(200, g.n - 1)]),
    }
    for what, vs in requests.items():
        o, ids = lg.decode_neighbors(h, torch.from_numpy(vs.astype(np.int32)).cuda(), "sorted")
        want = np.concatenate([col[off[v]:off[v + 1]] for v in vs])
        assert np.array_equal(o.cpu().numpy(), np.concatenate([[0], np.cumsum(np.diff(off)[vs])])), what
        assert np.array_equal(ids.cpu().numpy(), want), what
    h.free()
