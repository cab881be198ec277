"""Sorted decodes of relabeled graphs: list lengths at the edges of the wave
sort's sizes and of the switch to a workgroup's (1,024).  Whole numbers: equal
to the input's lists."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025, 2047, 2048, 2049, 4095,
         4097]


@pytest.mark.parametrize("enc", [dict(ids="local", offsets="ef", relabel=True), dict(layout="plain", relabel="greedy"),
                                 dict(ids="varint-diff", relabel=True), dict(ids="local-gap", relabel="greedy")],
                         ids=["local-dm", "plain-greedy", "varint-dm", "gap-greedy"])
def test_sizes(enc):
    n = 30000
    rng = np.random.default_rng(6)
    src = np.concatenate([np.full(d, i) for i, d in enumerate(SIZES)])
    dst = np.concatenate([rng.choice(np.arange(100, n), d, replace=False) for d in SIZES])
    g = gg.canonical_csr(n, torch.from_numpy(src), torch.from_numpy(dst))
    off, col = g.numpy()
    assert np.diff(off)[: len(SIZES)].tolist() == SIZES
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **enc)
    for vs in (np.arange(len(SIZES)), rng.permutation(np.repeat(np.arange(len(SIZES)), 60)), np.array([16])):
        o, ids = lg.decode_neighbors(h, torch.from_numpy(vs.astype(np.int32)).cuda(), "sorted")
        want = np.concatenate([col[off[v]:off[v + 1]] for v in vs])
        assert np.array_equal(o.cpu().numpy(), np.concatenate([[0], np.cumsum(np.diff(off)[vs])]))
        assert np.array_equal(ids.cpu().numpy(), want)
    h.free()
