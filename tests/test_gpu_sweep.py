"""The row sweeps of cfpq_closure (sweep.h): every rule kind -- pulled (fixed
left operand), scattered (fixed right operand), both fixed, both growing --
heads that are scatter targets and sources at once, initial bits on growing
nonterminals, at sizes around the row-word and wavefront edges, against the
oracle bit for bit."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import graphs, grammars
from workloads.grammars import CNF

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def _g(name, nts, term, rules):
    ix = {x: i for i, x in enumerate(nts)}
    ts = ("a", "b")
    return CNF(tuple(nts), ts, tuple((ix[h], ts.index(x)) for h, x in term),
               tuple((ix[h], ix[l], ix[r]) for h, l, r in rules), name)


GRAMMARS = [
    grammars.anbn(), grammars.dyck(), grammars.transitive_closure(),
    # a+ b, left-linear: S is source and target of a scatter, with initial bits
    _g("left_linear", ["S", "A", "B"], [("S", "a"), ("A", "a"), ("B", "b")], [("S", "S", "A"), ("S", "S", "B")]),
    _g("right_linear", ["S", "A", "B"], [("S", "b"), ("A", "a"), ("B", "b")], [("S", "A", "S"), ("S", "B", "S")]),
    # chains of scatters (X from S, Y from X, S from Y), pulls into targets, a terminal rule given twice
    _g("scatter_chain", ["S", "X", "Y", "A", "B"], [("S", "a"), ("A", "a"), ("B", "b"), ("A", "a"), ("X", "b")],
       [("X", "S", "B"), ("Y", "X", "A"), ("S", "Y", "B"), ("X", "A", "Y"), ("Y", "A", "B")]),
    # several growing pairs with one head, and a growing pair whose operands start empty
    _g("pairs", ["S", "X", "Y", "A", "B"], [("A", "a"), ("B", "b"), ("X", "a")],
       [("S", "X", "Y"), ("S", "Y", "X"), ("X", "A", "X"), ("Y", "A", "B"), ("Y", "S", "B")]),
]


def _check(cfpq, n, e, g, **kw):
    print("[gpu-case] sweep", g.name, n, len(e), kw, file=sys.stderr, flush=True)
    want = worklist.closure(n, e, g)
    res = cfpq.closure(n, e, g, **kw)
    assert res.stats["converged"] == 1
    assert np.array_equal(cfpq.result_bits(res), want)
    assert not res.bits[:, n:].any()
    return res


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
@pytest.mark.parametrize("n", [513, 640, 1023, 1500, 4090])
def test_sweep_equals_oracle(cfpq, g, n):
    if n > 2000 and g.name not in ("anbn", "scatter_chain", "left_linear"):
        n = 2049  # the oracle's worklist takes minutes on dense closures of that size
    _, e = graphs.erdos_renyi(n, 3 * n // 2, 300 + n, labels=2)
    _check(cfpq, n, e, g)


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
def test_sweep_of_hosted_products(cfpq, g):
    """Padded sides from 4096 on: products over growing pairs chosen per loop."""
    n = 4200
    _, e = graphs.erdos_renyi(n, int(0.9 * n), 77, labels=2)
    _check(cfpq, n, e, g)


@pytest.mark.parametrize("n", [5000, 8192, 9000, 16384, 16385])
def test_sweep_of_wide_rows(cfpq, n):
    """Two and four row words a lane, 32 and 64 rows a workgroup, few and many
    bits a row (scattered one by one, or turned in LDS); one node more takes
    the product loops."""
    _, e = graphs.erdos_renyi(n, n, 78, labels=2)
    _check(cfpq, n, e, grammars.anbn())
    # dense: against the product loops, whose closures the oracle covers at sizes it can take
    _, e = graphs.erdos_renyi(n, 4 * n, 79, labels=2)
    print("[gpu-case] sweep against the dense products", n, file=sys.stderr, flush=True)
    a = cfpq.closure(n, e, grammars.anbn())
    b = cfpq.closure(n, e, grammars.anbn(), path="fp4", hybrid=0)
    assert bool((a.bits == b.bits).all())


def test_sweep_hub_multi_edges_and_no_edges(cfpq):
    import torch
    n = 700
    hub = [(0, 0, j) for j in range(1, n)] + [(j, 1, 0) for j in range(1, n, 2)] + [(3, 0, 3), (3, 1, 3)] * 3
    e = np.asarray(hub, np.int32)
    for g in (grammars.anbn(), GRAMMARS[3], GRAMMARS[5], grammars.dyck()):
        _check(cfpq, n, e, g)
    # lists past the wavefront's and the workgroup's share on both ends
    both = np.asarray([(0, 0, j) for j in range(1, n)] + [(j, 0, (7 * j) % n) for j in range(1, n)]
                      + [(j, 1, 5) for j in range(n)] + [(5, 1, j) for j in range(0, n, 2)], np.int32)
    for g in (grammars.anbn(), GRAMMARS[5], grammars.dyck()):
        _check(cfpq, n, both, g)
    res = cfpq.closure(n, np.zeros((0, 3), np.int32), grammars.dyck())
    assert not res.bits.any() and res.stats["converged"] == 1 and res.stats["iterations"] == 1
    # device edges out of range are refused; more edges than the lists hold take the product loops
    bad = e.copy()
    bad[5, 2] = n
    with pytest.raises(cfpq.CfpqError) as ei:
        cfpq.closure(n, torch.from_numpy(bad).cuda(), grammars.anbn())
    assert ei.value.status == -1
    _, many = graphs.erdos_renyi(n, 17 * 768, 5, labels=2)
    _check(cfpq, n, many, grammars.anbn())


@pytest.mark.parametrize("n,iters", [(1000, 1), (1000, 5), (1000, 9), (4500, 3)])
def test_sweep_cut_short_is_sound(cfpq, n, iters):
    _, e = graphs.erdos_renyi(n, 3 * n, 43, labels=2)
    g = grammars.anbn()
    full = worklist.closure(n, e, g)
    res = cfpq.closure(n, e, g, max_iters=iters, allow_partial=True)
    got = cfpq.result_bits(res)
    assert not (got & ~full).any()
    if res.status == -4:
        assert res.stats["iterations"] == iters and res.stats["converged"] == 0
        assert got.any()


@pytest.mark.parametrize("n", [600, 4200])
def test_sweep_reads_nothing_stale_in_the_workspace(cfpq, n):
    """A growing pair whose right operand never changes while its left one
    does: the product must not read a transpose that was never made."""
    import torch
    g = _g("idle_right", ["S", "X", "Y", "A", "B"], [("A", "a"), ("B", "b")],
           [("X", "A", "B"), ("Y", "Y", "B"), ("S", "X", "Y"), ("S", "Y", "X")])
    _, e = graphs.erdos_renyi(n, 2 * n, 21, labels=2)
    _check(cfpq, n, e, g, workspace=torch.full((256 << 20,), 255, dtype=torch.uint8, device="cuda"))
