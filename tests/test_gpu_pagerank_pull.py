"""The pull and the Varint kernels over several iterations, on graphs and
iteration counts that propagation blocking does not serve: lists cut into
segments (above 4,096 entries) and byte chunks (above 8,192 bytes), of which
every iteration after the first reads what the one before wrote.

Tolerance: a vertex of d entries sums them in FP32 in at most d steps, each
rounding by 2^-24, and rounds three times more; after t iterations at most
t (d_max + 4) 2^-24 of a score.  Over the whole vector L1 1e-5, as for the
other kernels."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _hubs(n, degrees, seed):
    """Hubs of these degrees over all labels and short lists between the others."""
    rng = np.random.default_rng(seed)
    h = len(degrees)
    src = [np.full(d, i) for i, d in enumerate(degrees)] + [rng.integers(h, n, n)]
    dst = [rng.choice(np.arange(h, n), d, replace=False) for d in degrees] + [rng.integers(h, n, n)]
    return gg.canonical_csr(n, torch.from_numpy(np.concatenate(src)), torch.from_numpy(np.concatenate(dst)))


GRAPHS = {
    "hubs": lambda: _hubs(60000, [25000, 9000, 4097, 4096, 100, 65, 64], 1),
    "kron15": lambda: gg.kronecker(15, 16, seed=2),
    "n1023": lambda: _hubs(1023, [700, 65], 3),
}
ENCS = [(dict(ids="local", offsets="ef"), (2, 5)), (dict(ids="local", relabel=True), (2, 5)),
        (dict(ids="local-gap"), (2, 5)), (dict(ids="local-gap", offsets="ef", relabel="greedy"), (3, 5)),
        (dict(ids="varint-full"), (2, 9)), (dict(ids="varint-diff", offsets="ef", relabel=True), (2, 9)),
        (dict(ids="varint-diff", offsets="plain-bv"), (4,))]


@pytest.mark.parametrize("name", GRAPHS)
def test_pull(name):
    g = GRAPHS[name]()
    off, col = g.numpy()
    off, col = off.astype(np.uint64), col.view(np.uint32)
    d_max = int(np.diff(off.astype(np.int64)).max())
    for enc, counts in ENCS:
        lg.lib().lg_trim()
        h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **enc)
        before = h.info()["device_bytes"]
        for t in counts:
            pr = lg.pagerank(h, 0.85, t)
            assert torch.equal(pr, lg.pagerank(h, 0.85, t)), (enc, t)
            want = np.asarray(orc.pagerank(off, col, 0.85, t), dtype=np.float64)
            err = np.abs(pr.cpu().numpy().astype(np.float64) - want)
            assert (err <= t * (d_max + 4) * 2.0 ** -24 * want).all(), (enc, t, (err / want).max())
            assert err.sum() <= 1e-5, (enc, t)
        assert h.info()["device_bytes"] - before < 8 * g.m, enc  # (no tables were built)
        h.free()


@pytest.mark.parametrize("ids", ["varint-full", "varint-diff"])
def test_chunked_hub(ids):
    """A hub over many 4 KiB chunks with values of one to four bytes."""
    n = (1 << 21) + 300
    rng = np.random.default_rng(8)
    far = np.unique(rng.integers(1 << 21, n, size=3000))
    leaves = np.concatenate([np.arange(1, 20000), far])
    src = np.concatenate([np.zeros(len(leaves), np.int64), np.full(40, 5)])
    dst = np.concatenate([leaves, far[:40]])
    g = gg.canonical_csr(n, torch.from_numpy(src), torch.from_numpy(dst))
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, ids=ids, offsets="ef")
    before = h.info()["device_bytes"]
    for t in (2, 7):
        pr = lg.pagerank(h, 0.85, t).cpu().numpy().astype(np.float64)
        want = orc.pagerank(off.astype(np.uint64), col.view(np.uint32), 0.85, t)
        assert np.abs(pr - want).sum() <= 1e-5, t
    assert h.info()["device_bytes"] - before < 8 * g.m + 16 * n
    h.free()
