"""Sorted decodes of relabeled graphs: list lengths at the edges of the wave,
workgroup and bitmap sorts (63-65, 128, 8191-8193, one of 20,000), IDs in
several 2^20 ranges, request counts around the one-launch head (1,024; 64 for
Varint lists), repeated hubs, and a graph whose IDs span more ranges than the
bitmap sort takes.  Whole numbers: equal to the input's lists; the
allocation-free entry point gives the same."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _hubs(n, sizes, seed):
    """Vertex i < len(sizes) with exactly sizes[i] neighbours spread over the IDs, and a few random edges between
    the others."""
    rng = np.random.default_rng(seed)
    h = len(sizes)
    src, dst = [], []
    for i, d in enumerate(sizes):
        src.append(np.full(d, i))
        dst.append(rng.choice(np.arange(h, n), d, replace=False))
    src.append(rng.integers(h, n, n // 50))
    dst.append(rng.integers(h, n, n // 50))
    return gg.canonical_csr(n, torch.from_numpy(np.concatenate(src)), torch.from_numpy(np.concatenate(dst)))


GRAPHS = {
    "edges": lambda: _hubs(40000, [2, 16, 17, 32, 33, 63, 64, 65, 127, 128, 129, 4096, 4097, 8191, 8192], 1),
    "long": lambda: _hubs(60000, [8193, 20000, 64, 3000], 2),
    "ranges": lambda: _hubs((1 << 21) + 77, [9000, 30000, 500], 3),
    "many ranges": lambda: _hubs((17 << 20) + 5, [9000, 100], 4),
    "kron14": lambda: gg.kronecker(14, 16, seed=5),
}
ENCS = [dict(ids="local", offsets="ef", relabel=True), dict(layout="plain", relabel="greedy"),
        dict(ids="varint-diff", offsets="ef", relabel=True)]


@pytest.mark.parametrize("enc", ENCS, ids=lambda e: "-".join(map(str, e.values())))
@pytest.mark.parametrize("name", GRAPHS)
def test_sorted(name, enc):
    g = GRAPHS[name]()
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **enc)
    rng = np.random.default_rng(7)
    for vs in (np.arange(20), np.repeat([0, 1, 2], 3), rng.integers(0, g.n, 63), rng.integers(0, g.n, 65),
               rng.integers(0, 40, 1024), rng.integers(0, g.n, 1025), rng.permutation(g.n)[:50000]):
        t = torch.from_numpy(vs.astype(np.int32)).cuda()
        o, ids = lg.decode_neighbors(h, t, "sorted")
        want = np.concatenate([col[off[v]:off[v + 1]] for v in vs])
        assert np.array_equal(o.cpu().numpy(), np.concatenate([[0], np.cumsum(np.diff(off)[vs])]))
        assert np.array_equal(ids.cpu().numpy(), want)
        if len(want) <= lg.LG_NOALLOC_MAX_SORTED_IDS:
            o2, ids2 = torch.empty_like(o), torch.empty(max(len(want), 1), dtype=torch.int32, device="cuda")
            assert lg.decode_neighbors_noalloc(h, t, o2, ids2, "sorted") == lg.LG_OK
            assert torch.equal(o, o2) and torch.equal(ids, ids2[:len(want)])
    h.free()


def test_missing_vertex():
    g = gg.kronecker(10, 16, seed=5)
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, relabel=True)
    for k in (1, 1024, 1025):
        vs = torch.zeros(k, dtype=torch.int32, device="cuda")
        vs[k - 1] = g.n
        with pytest.raises(lg.LGError) as e:
            lg.decode_neighbors(h, vs)
        assert e.value.status == lg.LG_ERR_INVALID
        vs[k - 1] = 1  # and the next call is sound again
        lg.decode_neighbors(h, vs)
    h.free()
