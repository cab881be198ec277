"""Batched searches whose levels change their ways: chains (levels of a vertex
or two), cliques strung on chains (every clique turns the search bottom-up and
back), a wide frontier that stays top-down (leaves beside a dense part it does
not reach), strips, and small searches by the same code.  Whole numbers: equal
to the oracle's."""

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu


def _path(n):
    return gg.csr_from_edges(n, [(i, i + 1) for i in range(n - 1)])


def _beads(count, clique, gap):
    edges, at, last = [], 0, None
    for _ in range(count):
        if last is not None:
            for i in range(gap):
                edges.append((last if i == 0 else at - 1, at))
                at += 1
            edges.append((at - 1, at))
        edges += [(at + i, at + j) for i in range(clique) for j in range(i)]
        at += clique
        last = at - 1
    return gg.csr_from_edges(at, edges)


def _leaves_beside_dense(leaves, dense):
    edges = [(0, i) for i in range(1, leaves)] + [(leaves - 1, leaves), (leaves, leaves + 1)]
    base = leaves + 2
    edges += [(base + i, base + j) for i in range(dense) for j in range(i)]
    return gg.csr_from_edges(base + dense, edges)


def _strip(w, h):
    edges = [(y * w + x, y * w + x + 1) for y in range(h) for x in range(w - 1)]
    edges += [(y * w + x, y * w + w + x) for y in range(h - 1) for x in range(w)]
    return gg.csr_from_edges(w * h, edges)


GRAPHS = [lambda: _path(3001), lambda: _beads(6, 70, 40), lambda: _beads(3, 200, 300),
          lambda: _leaves_beside_dense(3000, 400), lambda: _strip(7, 400), lambda: gg.kronecker(11, 8, seed=2)]
ENCS = [dict(), dict(ids="local", offsets="ef"), dict(layout="plain"), dict(ids="local-gap"), dict(ids="varint-diff")]


@pytest.mark.parametrize("enc", ENCS, ids=lambda e: "-".join(map(str, e.values())) or "global")
@pytest.mark.parametrize("autotune", [False, True])
def test_batches(enc, autotune):
    gs = [f() for f in GRAPHS]
    hs = [lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **enc) for g in gs]
    jobs = [(i, r) for i, g in enumerate(gs) for r in (0, g.n // 2, g.n - 1)]
    for max_depth in (-1, 45):
        plan = lg.BatchPlan(hs, jobs, max_depth=max_depth, autotune=autotune)
        plan.depth_flat.fill_(-7)
        plan.parent_flat.fill_(-7)
        plan.run()
        torch.cuda.synchronize()
        for i, (k, r) in enumerate(jobs):
            off, col = gs[k].numpy()
            d0, p0 = orc.bfs(off, col, r, max_depth=max_depth)
            assert np.array_equal(plan.depth(i).cpu().numpy(), d0), (k, r, max_depth)
            assert np.array_equal(plan.parent(i).cpu().numpy(), p0), (k, r, max_depth)
        plan.free()
    for h in hs:
        h.free()


@pytest.mark.parametrize("enc", ENCS, ids=lambda e: "-".join(map(str, e.values())) or "global")
def test_small_searches(enc):
    for f in GRAPHS:
        g = f()
        off, col = g.numpy()
        h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, **enc)
        roots = [0, g.n // 2, g.n - 1]
        d, p = lg.bfs(h, roots)
        for i, r in enumerate(roots):
            d0, p0 = orc.bfs(off, col, r)
            assert np.array_equal(d[i].cpu().numpy(), d0) and np.array_equal(p[i].cpu().numpy(), p0), (g.n, r)
        h.free()
