"""Neighbor queries on relabeled graphs under budgets that hold what the sort
of their lists takes and little more: nothing beside the lists up to 8,192
entries, a copy of them above, the buffers of the radix sort where the IDs
span more than 16 ranges of 2^20.  The lists are whole numbers: equal to the
input."""

import numpy as np
import pytest
import torch

from paper_2010_15879_amd import graphgen as gg
from paper_2010_15879_amd import lg

pytestmark = pytest.mark.gpu

SLACK = 8192


def _hub(n, degree):
    return gg.canonical_csr(n, torch.zeros(degree, dtype=torch.int64), torch.arange(1, degree + 1) * (n // (degree + 1)))


@pytest.mark.parametrize("n,degree,per_id,fits", [
    (60000, 5000, 4, True), (60000, 8192, 4, True), (60000, 8193, 8, True), (60000, 20000, 8, True),
    (60000, 20000, 6, False), ((17 << 20) + 5, 9000, 12, False), ((17 << 20) + 5, 9000, 28, True)])
def test_budget_of_a_hub(n, degree, per_id, fits):
    g = _hub(n, degree)
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, relabel=True)
    resident = h.info()["device_bytes"]
    budget = resident + per_id * degree + SLACK + (40000 if per_id == 28 else 0)
    srv = lg.Server([h], budget_bytes=budget, workers=1)
    r = srv.wait(srv.submit("neighbors", 0, 0))
    st = srv.stats()
    srv.free()
    assert (r["status"] == lg.LG_OK) == fits
    assert st["overruns"] == 0 and st["peak_bytes"] <= budget
    if fits:
        assert np.array_equal(r["ids"], col[off[0]:off[1]].astype(np.uint32))
    h.free()


def test_batches_in_turn():
    """Short and long batches one after the other on the same worker."""
    g = _hub(60000, 12000)
    off, col = g.numpy()
    h = lg.encode(g.row_offsets.cuda(), g.col.cuda(), g.n, ids="local", offsets="ef", relabel="greedy")
    srv = lg.Server([h], workers=1, max_batch=8)
    vs = [0] + [int(x) for x in col[:20]] + [0, 0, 59999, 0] + [int(x) for x in col[20:60]]
    tickets = [srv.submit("neighbors", 0, v) for v in vs]
    for v, t in zip(vs, tickets):
        r = srv.wait(t)
        assert r["status"] == lg.LG_OK
        assert np.array_equal(r["ids"], col[off[v]:off[v + 1]].astype(np.uint32)), v
    assert srv.stats()["overruns"] == 0
    srv.free()
    h.free()
