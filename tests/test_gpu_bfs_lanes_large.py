"""Calls of a few roots on graphs above 2^14 vertices, which run on the
device's lanes: every row equals the call with its root alone and the
oracle's, work on the caller's stream is ordered around the call, and two
threads may call at once, one with lanes and one with a multi-source batch.
One root of the in-order kernels (gap, Varint) with levels in both
directions.  Whole numbers."""

import threading

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

ENCS = [dict(), dict(ids="local", offsets="ef", relabel=True), dict(layout="plain", relabel="greedy"),
        dict(ids="local-gap"), dict(ids="local-gap", offsets="ef", relabel=True),
        dict(ids="varint-full", offsets="ef", relabel="greedy"), dict(ids="varint-diff")]
IDS = ["-".join(map(str, e.values())) or "global" for e in ENCS]


def _graph(name):
    if name == "kron15":
        return gg.kronecker(15, 16, seed=5, device="cuda")
    if name == "er15":
        return gg.erdos_renyi(15, 8, seed=3, device="cuda")
    i = torch.arange(200 * 100, device="cuda").view(200, 100)  # a grid: a hundred levels and more
    return gg.canonical_csr(i.numel(), torch.cat([i[:, :-1].reshape(-1), i[:-1].reshape(-1)]),
                            torch.cat([i[:, 1:].reshape(-1), i[1:].reshape(-1)]))


@pytest.mark.parametrize("enc", ENCS, ids=IDS)
@pytest.mark.parametrize("name", ["kron15", "er15", "grid"])
def test_nine_roots(name, enc):
    g = _graph(name)
    off, col = g.numpy()
    h = lg.encode(g.row_offsets, g.col, g.n, **enc)
    roots = gg.pick_roots(g, 9, seed=2)
    for max_depth in (-1, 3):
        d_all, p_all = lg.bfs(h, roots, max_depth=max_depth)
        for i, r in enumerate(roots):
            d1, p1 = lg.bfs(h, [r], max_depth=max_depth)
            assert torch.equal(d_all[i], d1[0]) and torch.equal(p_all[i], p1[0]), (i, r)
        for i in (0, 8):
            d0, p0 = orc.bfs(off.astype(np.uint64), col.view(np.uint32), roots[i], max_depth=max_depth)
            assert np.array_equal(d_all[i].cpu().numpy(), d0), (i, max_depth)
            if not enc.get("relabel"):
                assert np.array_equal(p_all[i].cpu().numpy(), p0), (i, max_depth)
            else:
                _, p2 = lg.bfs(h, [roots[i]], max_depth=max_depth, mode="td")
                assert torch.equal(p_all[i], p2[0]), (i, max_depth)
    h.free()


@pytest.mark.parametrize("enc", [ENCS[0], ENCS[4]], ids=["global", "gap-dm"])
def test_stream_order(enc):
    g = _graph("kron15")
    h = lg.encode(g.row_offsets, g.col, g.n, **enc)
    roots = gg.pick_roots(g, 9, seed=3)
    ref, _ = lg.bfs(h, roots)
    torch.cuda.synchronize()
    for _ in range(3):
        depth = torch.empty((len(roots), g.n), dtype=torch.int32, device="cuda")
        parent = torch.empty_like(depth)
        depth.fill_(123)
        lg.bfs(h, roots, depth_out=depth, parent_out=parent)
        total = depth.sum()
        assert torch.equal(depth, ref) and int(total) == int(ref.sum())
    h.free()


def test_two_threads():
    graphs = [_graph("kron15"), _graph("er15")]
    hs = [lg.encode(g.row_offsets, g.col, g.n) for g in graphs]
    roots = [gg.pick_roots(g, c, seed=5) for g, c in zip(graphs, (9, 40))]
    ref = [lg.bfs(h, r) for h, r in zip(hs, roots)]
    torch.cuda.synchronize()
    out, errors = [[], []], []

    def work(i):
        try:
            s = torch.cuda.Stream()
            for _ in range(6):
                with torch.cuda.stream(s):
                    got = lg.bfs(hs[i], roots[i], stream=s)
                s.synchronize()
                out[i].append(got)
        except Exception as e:  # surfaced below
            errors.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(2)]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errors, errors
    for i in range(2):
        assert len(out[i]) == 6
        for d, p in out[i]:
            assert torch.equal(d, ref[i][0]) and torch.equal(p, ref[i][1]), i
    for h in hs:
        h.free()
