"""PageRank with damping next to 1, whose base term (1 - damping) / n vanishes:
scores then lie as low as 1 / (n d), below what fixed-point sums resolve, and
are summed in FP32.

A star's leaves hold damping / (n leaves) after one iteration, by three FP32
roundings (the contribution, the product and the sum with the base term):
within 3 units of 2^-24."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("enc", [dict(relabel=True), dict(layout="plain", relabel="greedy"),
                                 dict(ids="local", offsets="ef", relabel=True)],
                         ids=["global-dm", "plain-greedy", "local-dm"])
def test_leaves_of_a_star(enc):
    n = 5000011
    g = gg.canonical_csr(n, torch.zeros(n - 1, dtype=torch.int64, device="cuda"),
                         torch.arange(1, n, device="cuda"))
    h = lg.encode(g.row_offsets, g.col, g.n, **enc)
    for damping in (1.0, float(np.float32(1.0 - 2.0 ** -24))):
        pr = lg.pagerank(h, damping, 1).cpu().numpy().astype(np.float64)
        want = (1.0 - damping) / n + damping / n / (n - 1)
        assert np.abs(pr[1:] - want).max() <= 3 * 2.0 ** -24 * want, (damping, pr[1], want)
    h.free()


@pytest.mark.parametrize("n,damping,kept", [(1 << 14, 0.85, True), (1 << 14, 1.0, True), (1 << 19, 0.85, True),
                                            (1 << 19, 1.0, False), (1 << 19, 0.99, True)])
def test_entry_buffers(n, damping, kept):
    """Which sums a call takes shows in what stays with the graph: the entry
    buffers of the exact sums, 8 bytes an entry.  (A star's scores go down to
    1 / (n (n - 1)).)"""
    lg.lib().lg_trim()
    g = gg.canonical_csr(n, torch.zeros(n - 1, dtype=torch.int64, device="cuda"), torch.arange(1, n, device="cuda"))
    h = lg.encode(g.row_offsets, g.col, g.n, relabel=True)
    before = h.info()["device_bytes"]
    lg.pagerank(h, damping, 20)
    assert (h.info()["device_bytes"] - before >= 8 * g.m) == kept
    h.free()
