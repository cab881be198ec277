"""Binned top-down levels: frontiers of short lists (more than 2,048 rows in a
tile of 8,192 edges), vertex counts on both sides of the wider bins (2^26),
relabeled parents, and the buffers of the claims, which belong to the device
and not to a graph: searches of several threads and graphs, lg_trim between.

A root tied to L leaves, every leaf to one of the vertices after them, beside
a dense part that the search does not reach: depths are 0, 1 and 2, and the
parent of a second-level vertex is the smallest label among its leaves."""

import threading

import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _graph(n, leaves, second, dense_edges, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    leaf = torch.arange(1, leaves + 1, device="cuda")
    to = torch.randint(leaves + 1, leaves + 1 + second, (leaves,), generator=gen, device="cuda")
    base = leaves + 1 + second
    rest = n - base
    a = torch.randint(0, rest, (dense_edges,), generator=gen, device="cuda") + base
    b = torch.randint(0, rest, (dense_edges,), generator=gen, device="cuda") + base
    g = gg.canonical_csr(n, torch.cat([torch.zeros_like(leaf), leaf, a]), torch.cat([leaf, to, b]))
    depth = torch.full((n,), -1, dtype=torch.int32, device="cuda")
    depth[0] = 0
    depth[1:leaves + 1] = 1
    depth[to] = 2
    parent = torch.full((n,), n, dtype=torch.int64, device="cuda")
    parent.scatter_reduce_(0, to, leaf, "amin")
    parent[parent == n] = -1
    parent[:leaves + 1] = 0
    return g, depth, parent.to(torch.int32)


def _binned(search):
    lg.prof_enable(True)
    lg.prof_reset()
    out = search()
    torch.cuda.synchronize()
    levels = lg.prof_query("td_bin_kernel")[0]
    lg.prof_enable(False)
    return out, levels


@pytest.mark.parametrize("size", ["2^21", "2^26"])
def test_short_rows(size):
    n, leaves, second, dense = ((1 << 21) + 77, 700000, 400000, 46000000) if size == "2^21" else \
        ((1 << 26) + 1000, 8600000, 5000000, 140000000)
    g, depth, parent = _graph(n, leaves, second, dense, 3)
    encs = [dict(layout="plain"), dict(ids="local", offsets="ef", relabel="degree")]
    for enc in encs + ([dict(), dict(relabel="greedy")] if size == "2^21" else []):
        h = lg.encode(g.row_offsets, g.col, g.n, **enc)
        (d, p), levels = _binned(lambda: lg.bfs(h, [0]))
        assert levels == 1, enc
        assert torch.equal(d[0], depth), enc
        if "relabel" not in enc:
            assert torch.equal(p[0], parent), enc
        else:
            d1, p1 = lg.bfs(h, [0], mode="td")
            assert torch.equal(d1, d) and torch.equal(p1, p), enc
        (d, _), levels = _binned(lambda: lg.bfs(h, [0], parent=False))
        assert levels == 1 and torch.equal(d[0], depth), enc
        h.free()
    lg.lib().lg_trim()


def test_claims_belong_to_the_device():
    made = [_graph((1 << 21) + 77 + 64 * i, 600000 + 20000 * i, 300000, 46000000, i) for i in range(3)]
    hs = [lg.encode(g.row_offsets, g.col, g.n) for g, _, _ in made]
    for (g, depth, _), h in zip(made, hs):
        before = h.info()["device_bytes"]
        (d, _), levels = _binned(lambda: lg.bfs(h, [0]))
        assert levels == 1 and torch.equal(d[0], depth)
        # the workspace of a search: at most 40 bytes a vertex, and 16 of the sweeps' tables
        assert h.info()["device_bytes"] - before <= 56 * g.n
    out, errors = [None] * len(hs), []

    def work(i):
        try:
            s = torch.cuda.Stream()
            got = []
            for turn in range(3):
                with torch.cuda.stream(s):
                    got.append(lg.bfs(hs[i], [0], stream=s))
                s.synchronize()
            out[i] = got
        except Exception as e:  # surfaced below
            errors.append(e)

    th = [threading.Thread(target=work, args=(i,)) for i in range(len(hs))]
    for t in th:
        t.start()
    for t in th:
        t.join()
    assert not errors, errors
    for got, (_, depth, parent) in zip(out, made):
        for d, p in got:
            assert torch.equal(d[0], depth) and torch.equal(p[0], parent)
    lg.lib().lg_trim()
    d, p = lg.bfs(hs[0], [0])
    assert torch.equal(d[0], made[0][1]) and torch.equal(p[0], made[0][2])
    for h in hs:
        h.free()
