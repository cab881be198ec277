"""Multi-source searches on a relabeled graph when the label-space cells do
not fit into memory, from the first level or when a search deeper than a byte
widens them: the rows equal those of the same call with room.  The device is
filled up to 0.5 and 1.1 GiB, where the cells take 0.63 GiB and the wide ones
0.5 more."""

import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

WIDTH, HEIGHT, DEPTH = 64, 1 << 15, 300


@pytest.fixture(scope="module")
def strip():
    v = torch.arange(WIDTH * HEIGHT, device="cuda").view(HEIGHT, WIDTH)
    g = gg.canonical_csr(v.numel(), torch.cat([v[:, :-1].reshape(-1), v[:-1].reshape(-1)]),
                         torch.cat([v[:, 1:].reshape(-1), v[1:].reshape(-1)]))
    h = lg.encode(g.row_offsets, g.col, g.n, ids="local", offsets="ef", relabel=True)
    roots = [(i * 52361) % g.n for i in range(40)]
    want = lg.bfs(h, roots, max_depth=DEPTH)
    assert int(want[0].max()) == DEPTH
    yield h, roots, want
    h.free()
    lg.lib().lg_trim()


def _fill(left):
    """Holds device memory until `left` bytes are free."""
    lg.lib().lg_trim()
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    while True:
        free = torch.cuda.mem_get_info()[0]
        if free <= left + (8 << 20):
            return held
        held.append(torch.empty(min(free - left, 64 << 30), dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("left", [1 << 29, 1181 << 20])
def test_cells_without_memory(strip, left):
    h, roots, (d0, p0) = strip
    d, p = torch.empty_like(d0), torch.empty_like(p0)
    held = _fill(left)
    try:
        lg.bfs(h, roots, max_depth=DEPTH, depth_out=d, parent_out=p)
        torch.cuda.synchronize()
    finally:
        del held
        torch.cuda.empty_cache()
    assert torch.equal(d, d0) and torch.equal(p, p0)
    d.fill_(-9)
    lg.bfs(h, roots, max_depth=DEPTH, depth_out=d, parent_out=p)  # and with room again
    assert torch.equal(d, d0) and torch.equal(p, p0)
