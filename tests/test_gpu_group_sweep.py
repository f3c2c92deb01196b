"""Batches whose instances run as group sweeps (513 to 4096 nodes) against the
oracle, and against the batch's dense products where the oracle is slow."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import graphs, grammars

from tests.test_gpu_sweep import GRAMMARS, _g

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def _poisoned(cfpq, items, **kw):
    """The batch with every workspace byte set beforehand."""
    import torch
    ws = torch.full((1 << 30,), 255, dtype=torch.uint8, device="cuda")
    return cfpq.batch_closure(items, workspace=ws, **kw)


IDLE = _g("idle_right", ["S", "X", "Y", "A", "B"], [("A", "a"), ("B", "b")],
          [("X", "A", "B"), ("Y", "Y", "B"), ("S", "X", "Y"), ("S", "Y", "X")])


@pytest.mark.parametrize("g", GRAMMARS + [IDLE], ids=lambda g: g.name)
def test_group_equals_oracle(cfpq, g):
    """Row widths on both sides of 16 lanes, ragged last row groups, sparse
    graphs and one dense enough for the turned scatter, beside instances of
    the other routes."""
    items = []
    for n, m in ((513, 700), (767, 1150), (1024, 1500), (1025, 1500), (1300, 1900), (600, 2400), (200, 400), (64, 90)):
        items.append((n, graphs.erdos_renyi(n, m, 900 + n, labels=2)[1], g))
    print("[gpu-case] group", g.name, file=sys.stderr, flush=True)
    for (n, e, _), res in zip(items, _poisoned(cfpq, items)):
        assert np.array_equal(cfpq.result_bits(res), worklist.closure(n, e, g)), n
        assert not res.bits[:, n:].any()
        assert res.stats["converged"] == 1


@pytest.mark.parametrize("g", [grammars.anbn(), grammars.dyck(), GRAMMARS[5]], ids=lambda g: g.name)
def test_group_equals_dense_products(cfpq, g):
    """Wide rows, 2048 to 4096 nodes and the first size past them, dense."""
    items = [(n, graphs.erdos_renyi(n, 3 * n, 31 + n, labels=2)[1], g) for n in (2048, 2049, 3000, 4095, 4096, 4097)]
    print("[gpu-case] group dense", g.name, file=sys.stderr, flush=True)
    for a, b in zip(_poisoned(cfpq, items), cfpq.batch_closure(items, hybrid=0)):
        assert bool((a.bits == b.bits).all()), a.n


def test_group_hubs_bad_edges_and_no_edges(cfpq):
    import torch
    n = 700
    both = np.asarray([(0, 0, j) for j in range(1, n)] + [(j, 0, (7 * j) % n) for j in range(1, n)]
                      + [(j, 1, 5) for j in range(n)] + [(5, 1, j) for j in range(0, n, 2)]
                      + [(3, 0, 3), (3, 1, 3)] * 3, np.int32)
    items = [(n, both, g) for g in (grammars.anbn(), GRAMMARS[3], GRAMMARS[5], grammars.dyck())]
    items.append((n, np.zeros((0, 3), np.int32), grammars.dyck()))
    print("[gpu-case] group hubs", file=sys.stderr, flush=True)
    for (_, e, g), res in zip(items, _poisoned(cfpq, items)):
        assert np.array_equal(cfpq.result_bits(res), worklist.closure(n, e, g))
    bad = both.copy()
    bad[5, 2] = n
    with pytest.raises(cfpq.CfpqError) as ei:
        cfpq.batch_closure([(n, torch.from_numpy(bad).cuda(), grammars.anbn())])
    assert ei.value.status == -1


@pytest.mark.parametrize("iters", [1, 2, 5])
def test_group_cut_short_is_sound(cfpq, iters):
    g = grammars.anbn()
    items = [(n, graphs.erdos_renyi(n, 3 * n, 43, labels=2)[1], g) for n in (600, 1000)]
    print("[gpu-case] group cut short", iters, file=sys.stderr, flush=True)
    for (n, e, _), res in zip(items, _poisoned(cfpq, items, max_iters=iters, allow_partial=True)):
        want = worklist.closure(n, e, g)
        got = cfpq.result_bits(res)
        assert res.status == -4 and res.stats["converged"] == 0 and res.stats["iterations"] == iters
        assert np.array_equal(got | want, want) and not np.array_equal(got, want)


@pytest.mark.parametrize("budget", [1 << 30, 14 << 20])
def test_group_in_a_server(cfpq, budget):
    """Requests that join a running group, leave it in another order, and (the
    small arena) fall back to the engine when their workspace does not fit."""
    import torch
    rng = np.random.default_rng(5)
    items = []
    for q in range(24):
        n = int(rng.integers(513, 1400))
        e = graphs.erdos_renyi(n, int(rng.integers(1, 4)) * n, 60 + q, labels=2)[1]
        items.append((n, torch.from_numpy(e).cuda() if q % 2 else e, GRAMMARS[q % len(GRAMMARS)]))
    items.append((2200, graphs.erdos_renyi(2200, 2200, 90, labels=2)[1], grammars.anbn()))
    items.append((300, graphs.erdos_renyi(300, 600, 91, labels=2)[1], grammars.dyck()))
    print("[gpu-case] group server", budget, file=sys.stderr, flush=True)
    with cfpq.Server(hbm_budget=budget, max_slots=12, hybrid_lanes=0) as srv:
        for wave in (items[:3], items[3:], items[::-1]):
            tickets = [srv.submit(*it) for it in wave]
            for it, t in zip(wave, tickets):
                info = srv.wait(t)
                assert info["status"] == 0
                want = cfpq.closure(*it)
                assert bool((info["result"].bits == want.bits).all()), it[0]
