"""The staged conjunctive closure (one-conjunct rules first, the rules of
several conjuncts once at the end) against the oracle and, at sizes the oracle
is slow for, against the loop over all rules (a named dense kernel takes it)."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import conjunctive, worklist
from workloads import grammars, graphs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def _two_heads():
    """Two late heads, one of them also set by a terminal rule; conjuncts with
    an edge matrix on the left (ROWS), on the right (COLS) and on neither
    side; one conjunct twice in a rule and one rule twice."""
    return grammars._mk_conj(
        "two_heads", ["S", "U", "D", "D1", "A", "B"], ["a", "b"],
        [("A", "a"), ("B", "b"), ("U", "b")],
        [("S", [("D", "D"), ("D", "B")]), ("S", [("A", "D"), ("A", "D"), ("D", "D1")]),
         ("U", [("A", "B"), ("D", "B"), ("A", "D1")]), ("U", [("A", "B"), ("D", "B"), ("A", "D1")]),
         ("D", [("A", "B")]), ("D", [("A", "D1")]), ("D1", [("D", "B")]), ("D", [("D", "D")])])


def _feeds_back():
    """The head of a rule of two conjuncts is read by a rule: not staged."""
    return grammars._mk_conj(
        "feeds_back", ["S", "D", "A", "B"], ["a", "b"], [("A", "a"), ("B", "b")],
        [("S", [("A", "D"), ("D", "B")]), ("D", [("S", "A")]), ("D", [("A", "B")])])


GRAMMARS = {"dyck_and_anbn": grammars.dyck_and_anbn, "two_heads": _two_heads, "feeds_back": _feeds_back}


@pytest.mark.parametrize("grammar", sorted(GRAMMARS))
@pytest.mark.parametrize("n,m", [(1, 1), (65, 200), (255, 900), (300, 70000)])
def test_staged_matches_oracle(cfpq, grammar, n, m):
    g = GRAMMARS[grammar]()
    _, e = graphs.erdos_renyi(n, m, 3, labels=2)
    print("[gpu-case] staged", grammar, n, m, file=sys.stderr, flush=True)
    want, _ = conjunctive.closure(n, e, g)
    got = worklist.unpack(cfpq.result_bits(cfpq.conjunctive_closure(n, e, g)), n)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("grammar", sorted(GRAMMARS))
@pytest.mark.parametrize("n,degree", [(513, 3), (1030, 4), (4100, 2), (16384, 1), (16385, 1)])
def test_staged_matches_the_loop(cfpq, grammar, n, degree):
    import torch
    g = GRAMMARS[grammar]()
    _, e = graphs.erdos_renyi(n, degree * n, 9, labels=2)
    d = torch.from_numpy(e).cuda()
    print("[gpu-case] staged", grammar, n, degree, file=sys.stderr, flush=True)
    got = cfpq.conjunctive_closure(n, d, g)
    want = cfpq.conjunctive_closure(n, d, g, path="fp4")
    assert torch.equal(got.bits, want.bits)
