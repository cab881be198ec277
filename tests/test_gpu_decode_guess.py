"""Decodes without a capacity allocate a guess ahead: a result does not hold
on to a guess far beyond its size, and a guess that does not fit into memory
is done without.  The lists are whole numbers: the results equal the input."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def graph():
    """Half of the vertices in a dense part, the others with one neighbour or none."""
    n = 400000
    gen = torch.Generator(device="cuda").manual_seed(2)
    half = n // 2
    src = torch.cat([torch.randint(0, half, (40 * half,), generator=gen, device="cuda"),
                     torch.arange(half, n - 1001, 2, device="cuda")])
    dst = torch.cat([torch.randint(0, half, (40 * half,), generator=gen, device="cuda"),
                     torch.arange(half + 1, n - 1000, 2, device="cuda")])
    g = gg.canonical_csr(n, src, dst)
    h = lg.encode(g.row_offsets, g.col, g.n)
    yield g, h
    h.free()


def _check(g, h, vs):
    off, col = g.numpy()
    o, ids = lg.decode_neighbors(h, torch.from_numpy(vs.astype(np.int32)).cuda())
    want = np.concatenate([col[off[v]:off[v + 1]] for v in vs])
    assert np.array_equal(o.cpu().numpy(), np.concatenate([[0], np.cumsum(np.diff(off)[vs])]))
    assert np.array_equal(ids.cpu().numpy(), want)
    return ids


def test_small_results_are_small(graph):
    g, h = graph
    for vs in (np.arange(g.n // 2, g.n), np.arange(g.n - 1000, g.n), np.arange(g.n - 1010, g.n - 990)):
        ids = _check(g, h, vs)
        assert ids.untyped_storage().nbytes() <= 4 * (2 * ids.numel() + (1 << 16)), len(vs)


def test_guess_without_memory(graph, monkeypatch):
    g, h = graph
    vs = np.arange(g.n // 2 - 500, g.n)
    made = torch.empty

    def empty(*size, **kw):
        if size and isinstance(size[0], int) and size[0] > 1 << 20:
            raise torch.OutOfMemoryError("no room")
        return made(*size, **kw)

    monkeypatch.setattr(torch, "empty", empty)
    _check(g, h, vs)
