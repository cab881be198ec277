"""One-launch searches in flight side by side: calls return with their kernels
queued, so their workspaces must not be taken while an earlier search still
uses them -- from more streams than there are workspaces, from one stream,
and with lg_trim between.  Long chains keep a search running while others are queued.  Whole numbers:
equal to the same call made alone."""

import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _chain(n, step):
    """0 - step - 2 step - ... (mod n), n no multiple of the prime step."""
    return gg.csr_from_edges(n, [(i * step % n, (i + 1) * step % n) for i in range(n - 1)])


@pytest.fixture(scope="module")
def chains():
    out = []
    for i in range(12):
        n = 1021 + 101 * i
        g = _chain(n, 7 if n % 7 else 11)
        h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, relabel=(False, False, True, "greedy")[i % 4])
        roots = [0, n // 2, n - 1]
        want = lg.bfs(h, roots)
        torch.cuda.synchronize()
        out.append((h, roots, want))
    yield out
    for h, _, _ in out:
        h.free()


def test_more_streams_than_workspaces(chains):
    streams = [torch.cuda.Stream() for _ in chains]
    got = []
    for turn in range(2):
        for (h, roots, want), s in zip(chains, streams):
            with torch.cuda.stream(s):
                got.append((lg.bfs(h, roots), want))
        if turn == 0:
            lg.lib().lg_trim()
    torch.cuda.synchronize()
    for (d, p), want in got:
        assert torch.equal(d, want[0]) and torch.equal(p, want[1])


def test_queued_on_one_stream(chains):
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        got = [(lg.bfs(h, roots), want) for _ in range(3) for h, roots, want in chains]
    s.synchronize()
    for (d, p), want in got:
        assert torch.equal(d, want[0]) and torch.equal(p, want[1])
