"""Row sweeps of graphs without edges, and of small ones in workspaces whose
every 16-bit word is a node number (the lists' code for "no entry" is 0xFFFF, so
a workspace of ones cannot show a list entry that was never written).

Without edges every relation is empty.  There the workspace's words name a row
past the result, which lies at the front of a larger buffer of ones: a stale
entry taken for a node shows as bits, and stays inside the buffer."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import conjunctive, worklist
from workloads import grammars, graphs

from tests.test_gpu_sweep import GRAMMARS

pytestmark = pytest.mark.gpu

NO_EDGES = np.zeros((0, 3), np.int32)


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def _words(count, value):
    """A workspace of `count` 16-bit words, each `value`."""
    import torch
    signed = value - (1 << 16) if value >= 1 << 15 else value
    return torch.full((count,), signed, dtype=torch.int16, device="cuda").view(torch.uint8)


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
@pytest.mark.parametrize("n", [513, 700, 4200, 8193, 16384])
def test_sweep_without_edges(cfpq, g, n):
    import torch
    k, rows = g.n_nonterminals, cfpq.padded_rows(n)
    words = k * rows * cfpq.row_words(n)
    past = min(k * rows, 0xFFF0)  # a row number the 16-byte lists could hold
    buf = torch.full(((past + (k + 1) * rows) * cfpq.row_words(n),), -1, dtype=torch.int64, device="cuda")
    print("[gpu-case] sweep without edges", g.name, n, file=sys.stderr, flush=True)
    res = cfpq.closure(n, NO_EDGES, g, out=buf[:words], workspace=_words(1 << 29, past))
    assert res.stats["converged"] == 1 and res.stats["iterations"] == 1
    assert not res.bits.any()
    assert bool((buf[words:] == -1).all())


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
def test_other_routes_without_edges(cfpq, g):
    """The resident and the group sweep, a server's worker and its lanes."""
    items = [(n, NO_EDGES, g) for n in (1, 64, 300, 512, 513, 1030, 4096, 4200)]
    print("[gpu-case] no edges, batch", g.name, file=sys.stderr, flush=True)
    for item, res in zip(items, cfpq.batch_closure(items, workspace=_words(1 << 28, 1))):
        assert not res.bits.any(), item[0]
    print("[gpu-case] no edges, server", g.name, file=sys.stderr, flush=True)
    with cfpq.Server(hbm_budget=1 << 30) as srv:
        for item, t in [(item, srv.submit(*item)) for item in items]:
            info = srv.wait(t)
            assert info["status"] == 0 and not info["result"].bits.any(), item[0]


@pytest.mark.parametrize("n", [300, 513, 4200])
def test_staged_conjunctive_without_edges(cfpq, n):
    g = grammars._mk_conj("right_linear_and", ["S", "U", "A"], ["a"], [("A", "a"), ("U", "a")],
                          [("S", [("A", "U"), ("A", "A")]), ("U", [("A", "U")])])
    print("[gpu-case] no edges, conjunctive", n, file=sys.stderr, flush=True)
    assert not cfpq.conjunctive_closure(n, NO_EDGES, g).bits.any()
    if n == 300:
        _, e = graphs.erdos_renyi(n, 500, 4, labels=1)
        got = worklist.unpack(cfpq.result_bits(cfpq.conjunctive_closure(n, e, g)), n)
        assert np.array_equal(got, conjunctive.closure(n, e, g)[0])


@pytest.mark.parametrize("word", [0, 1, 300])
@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
def test_stale_words_that_are_nodes(cfpq, g, word):
    """Few edges, so that most lists stay empty."""
    for n, m in ((600, 90), (1030, 1500), (4200, 2100)):
        _, e = graphs.erdos_renyi(n, m, 50 + n, labels=2)
        print("[gpu-case] stale words", g.name, n, word, file=sys.stderr, flush=True)
        want = worklist.closure(n, e, g)
        assert np.array_equal(cfpq.result_bits(cfpq.closure(n, e, g, workspace=_words(1 << 28, word))), want)
        got, = cfpq.batch_closure([(n, e, g)], workspace=_words(1 << 28, word))
        assert np.array_equal(cfpq.result_bits(got), want)
