"""PageRank calls of a few iterations over large unrelabeled local IDs: as
accurate as over global IDs of the same graph, whose sums are exact.

Tolerance: an iteration rounds a contribution twice (score and quotient), the
score and the base term, each by 2^-24 of its value: after t iterations at
most (4 t + 2) 2^-24 of a score, plus the fixed-point unit 2^-61 per entry and
iteration."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _star(n, leaves, damping, iters):
    """Ranks of a hub, of a leaf and of an edgeless vertex, in 64 bits."""
    hub = leaf = lone = 1.0 / n
    for _ in range(iters):
        base = (1.0 - damping) / n + damping * lone * (n - 1 - leaves) / n
        hub, leaf, lone = base + damping * leaf * leaves, base + damping * hub / leaves, base
    return hub, leaf, lone


@pytest.mark.parametrize("offsets", ["packed", "ef"])
@pytest.mark.parametrize("iters", [1, 2, 5])
def test_star_of_local_ids(offsets, iters):
    n, leaves = (1 << 22) + 77, 4000000
    hub_of = torch.zeros(leaves, dtype=torch.int64, device="cuda")
    g = gg.canonical_csr(n, hub_of, torch.arange(1, leaves + 1, device="cuda"))
    h = lg.encode(g.row_offsets, g.col, g.n, ids="local", offsets=offsets)
    damping = float(np.float32(0.85))
    pr = lg.pagerank(h, damping, iters).cpu().numpy().astype(np.float64)
    h.free()
    hub, leaf, lone = _star(n, leaves, damping, iters)
    want = np.full(n, lone)
    want[1:leaves + 1] = leaf
    want[0] = hub
    deg = np.where(np.arange(n) == 0, leaves, 1)
    tol = (4 * iters + 2) * 2.0 ** -24 * want + iters * (deg + 1) * 2.0 ** -61
    off = np.abs(pr - want)
    assert (off <= tol).all(), (iters, (off / want).max() * 2 ** 24)
