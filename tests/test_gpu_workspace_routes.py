"""Workspaces and arenas that hold the product loops' matrices but not the row
sweeps': the closure runs as product loops, with the same bits."""
from __future__ import annotations

import ctypes
import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import grammars, graphs

from tests.test_gpu_sweep import _g

pytestmark = pytest.mark.gpu

# many growing nonterminals and pairs of them: the sweeps keep more matrices than the loops
WIDE = _g("wide", ["S", "T", "U", "V", "A", "B"],
          [("S", "b"), ("T", "a"), ("U", "a"), ("U", "b"), ("V", "a"), ("A", "a"), ("B", "b")],
          [("V", "U", "U"), ("B", "V", "V"), ("T", "U", "V"), ("U", "T", "S"), ("S", "S", "V"), ("U", "B", "U"),
           ("A", "T", "V")])


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def _bytes(cfpq, n, e, g, **kw):
    from paper_1707_01007_amd import _abi
    graph, keep_e = cfpq._graph_struct(n, e)
    gs, keep_g = cfpq._grammar_struct(g)
    size = ctypes.c_size_t(0)
    _abi.check(cfpq.lib().cfpq_workspace_bytes(ctypes.byref(graph), ctypes.byref(gs),
                                               ctypes.byref(cfpq._options(**kw)), ctypes.byref(size)))
    return size.value


@pytest.mark.parametrize("n,degree,g", [(600, 2, grammars.dyck()), (1500, 1, WIDE), (4200, 1, WIDE)],
                         ids=lambda x: getattr(x, "name", str(x)))
@pytest.mark.parametrize("sized_for", [{"warm_start": True}, {"profile": True}, {"path": "fp4"}], ids=str)
def test_workspace_sized_for_other_options(cfpq, n, degree, g, sized_for):
    import torch
    from paper_1707_01007_amd import _abi
    _, e = graphs.erdos_renyi(n, degree * n // 2, 5, labels=2)
    size = _bytes(cfpq, n, e, g, **sized_for)
    assert size < _bytes(cfpq, n, e, g)
    graph, keep_e = cfpq._graph_struct(n, e)
    gs, keep_g = cfpq._grammar_struct(g)
    want = worklist.closure(n, e, g)
    out = torch.empty(int(cfpq.lib().cfpq_result_bytes(n, g.n_nonterminals)) // 8, dtype=torch.int64, device="cuda")
    ws = torch.full((size,), 1, dtype=torch.uint8, device="cuda")
    stats = _abi.Stats()

    def call(nbytes):
        return cfpq.lib().cfpq_closure(ctypes.byref(graph), ctypes.byref(gs), ctypes.byref(cfpq._options()),
                                       cfpq._stream_ptr(None), ctypes.c_void_p(ws.data_ptr()), ctypes.c_size_t(nbytes),
                                       ctypes.c_void_p(out.data_ptr()), ctypes.byref(stats))

    print("[gpu-case] workspace of other options", g.name, n, sized_for, file=sys.stderr, flush=True)
    assert call(size) == 0 and stats.converged == 1
    bits = out.view(g.n_nonterminals, cfpq.padded_rows(n), cfpq.row_words(n))
    assert np.array_equal(cfpq.result_bits(cfpq.Result(n, g.n_nonterminals, bits, {}, 0)), want)
    assert call(size // 2) == _abi.CFPQ_ENOMEM


def test_lane_in_an_arena_too_small_for_the_sweeps(cfpq):
    n = 4000
    _, e = graphs.erdos_renyi(n, n // 2, 6, labels=2)
    loops, sweeps = _bytes(cfpq, n, e, WIDE, path="fp4"), _bytes(cfpq, n, e, WIDE)
    assert sweeps > loops + (4 << 20)
    want = worklist.closure(n, e, WIDE)
    for budget in (loops + (2 << 20), sweeps + (2 << 20)):
        print("[gpu-case] lane in a small arena", budget, file=sys.stderr, flush=True)
        with cfpq.Server(hbm_budget=budget, max_slots=1, hybrid_lanes=1) as srv:
            tickets = [srv.submit(n, e, WIDE) for _ in range(2)]
            for t in tickets:
                info = srv.wait(t)
                assert info["status"] == 0 and np.array_equal(cfpq.result_bits(info["result"]), want)
    with cfpq.Server(hbm_budget=loops // 2, max_slots=1, hybrid_lanes=1) as srv:
        with pytest.raises(cfpq.CfpqError) as ei:
            srv.submit(n, e, WIDE)
        assert ei.value.status == -2
