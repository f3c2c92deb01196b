"""Requests of 513 to 3840 nodes with rules over two growing operands, which take
idle lanes: alone, several together, beside large lane requests that fill the
arena, and with device edges out of range."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import grammars, graphs

from tests.test_gpu_sweep import GRAMMARS

pytestmark = pytest.mark.gpu

PAIRS = GRAMMARS[6]


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def _items(sizes, g, degree=1):
    return [(n, graphs.erdos_renyi(n, degree * n, 7 + n, labels=2)[1], g) for n in sizes]


def _serve(cfpq, srv, items, want):
    tickets = [srv.submit(*it) for it in items]
    for it, t in zip(items, tickets):
        info = srv.wait(t)
        assert info["status"] == 0
        assert np.array_equal(cfpq.result_bits(info["result"]), want[it[0], it[2].name]), (it[0], it[2].name)


@pytest.mark.parametrize("lanes", [0, 1, 2])
def test_requests_with_pairs(cfpq, lanes):
    items = _items((513, 600, 1024, 1025, 1500, 2100), grammars.dyck()) + _items((700, 1100, 2200), PAIRS) \
        + _items((1200,), PAIRS, 3) + _items((800, 1400), grammars.anbn()) + _items((300,), grammars.dyck())
    want = {(n, g.name): worklist.closure(n, e, g) for n, e, g in items}
    print("[gpu-case] serve pairs", lanes, file=sys.stderr, flush=True)
    with cfpq.Server(hbm_budget=1 << 30, max_slots=6, hybrid_lanes=lanes) as srv:
        for it in items:
            _serve(cfpq, srv, [it], want)
        for wave in (items, items[::-1], items[1::2] * 2):
            _serve(cfpq, srv, wave, want)


def test_small_arena_beside_large_requests(cfpq):
    """A large request that waits for nearly all of the arena is not kept from
    it by smaller ones queued behind it with their blocks."""
    large = _items((4100, 4200, 4300), grammars.anbn())
    mid = _items((600, 900, 1300, 1700), grammars.dyck())
    want = {(n, g.name): worklist.closure(n, e, g) for n, e, g in large + mid}
    order = [large[0], mid[0], large[1], mid[1], large[2], mid[2], mid[3], large[0], large[1], mid[0]]
    for budget in (34 << 20, 48 << 20, 96 << 20):
        print("[gpu-case] serve small arena", budget, file=sys.stderr, flush=True)
        with cfpq.Server(hbm_budget=budget, max_slots=4, hybrid_lanes=2) as srv:
            for _ in range(3):
                _serve(cfpq, srv, order, want)


def test_bad_device_edge_in_a_lane(cfpq):
    import torch
    n, e, g = _items((900,), grammars.dyck())[0]
    bad = e.copy()
    bad[7, 0] = n
    print("[gpu-case] serve bad edge", file=sys.stderr, flush=True)
    with cfpq.Server(hbm_budget=1 << 30) as srv:
        assert srv.wait(srv.submit(n, torch.from_numpy(bad).cuda(), g))["status"] == -1
        info = srv.wait(srv.submit(n, torch.from_numpy(e).cuda(), g))
        assert info["status"] == 0 and np.array_equal(cfpq.result_bits(info["result"]), worklist.closure(n, e, g))
