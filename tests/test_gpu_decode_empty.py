"""Decodes of requests made mostly of empty lists: single entries 63 to 257
lists apart, entries at the request's two ends alone, long runs of empty lists
before, between and after long ones, unit counts (lists plus entries) at the
edges of the pieces the output is cut into.  The lists are whole numbers: the
results equal the input."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

N = 70000
OPTS = [dict(ids="global", offsets="packed"), dict(ids="local", offsets="ef"), dict(layout="plain"),
        dict(ids="global", offsets="interleaved-bv"), dict(ids="local", offsets="ef", relabel=True)]


def _graph():
    """Vertices 0 .. 999 with 1 to 3 neighbours, 1000 with 5,000 of them, the rest edgeless."""
    rng = np.random.default_rng(3)
    edges = [(int(a), int(b)) for a, b in zip(rng.integers(0, 1000, 900), rng.integers(0, 1000, 900)) if a != b]
    edges += [(1000, 1001 + i) for i in range(5000)]
    return gg.csr_from_edges(N, edges)


@pytest.mark.parametrize("opts", OPTS, ids=lambda o: "-".join(map(str, o.values())))
def test_empty(opts):
    g = _graph()
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **opts)
    lone = N - 1
    short = np.nonzero(np.diff(off) == 1)[0][0]
    rng = np.random.default_rng(4)

    def apart(gap, count):
        vs = np.full(gap * count, lone)
        vs[gap // 2::gap] = rng.integers(0, 1000, count)
        return vs

    requests = [apart(gap, 700) for gap in (63, 64, 65, 100, 257)]
    requests += [np.concatenate([[short], np.full(k, lone), [short]]) for k in (1, 62, 63, 250, 252, 253, 1 << 20)]
    requests += [np.concatenate([np.full(3000, lone), [1000], np.full(1 << 18, lone), [1000, short], np.full(777, lone)]),
                 np.concatenate([[1000], np.full(100000, lone)]), np.concatenate([np.full(100000, lone), [1000]]),
                 np.full(5000, lone), np.concatenate([np.full(2047, lone), [short]])]
    for i, vs in enumerate(requests):
        o, ids = lg.decode_neighbors(h, torch.from_numpy(vs.astype(np.int32)).cuda(), "sorted")
        want = np.concatenate([col[off[v]:off[v + 1]] for v in vs[np.diff(off)[vs] > 0]] or [col[:0]])
        assert np.array_equal(o.cpu().numpy(), np.concatenate([[0], np.cumsum(np.diff(off)[vs])])), i
        assert np.array_equal(ids.cpu().numpy(), want), i
    h.free()
