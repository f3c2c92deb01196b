"""Small graphs at the densities where the resident sweep hands over to the
kernel that multiplies, and dense first loops, whose scatters run turned:
against the oracle, alone and in a batch."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import grammars

from tests.test_gpu_sweep import _g

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


AB = [("A", "a"), ("B", "b")]
GRAMMARS = [
    grammars.anbn(), grammars.dyck(),
    # initial bits on the scatters' operand beside a rule of two lists
    _g("right", ["S", "A", "B"], [("S", "a"), *AB], [("S", "A", "S")]),
    _g("seeded", ["S", "X", "A", "B"], [("S", "b"), *AB], [("S", "A", "X"), ("S", "A", "B"), ("X", "S", "B")]),
    # four heads (no room for turned operands at 512 nodes), with and without products
    _g("four", ["S", "X", "Y", "Z", "A", "B"], AB,
       [("S", "A", "X"), ("S", "A", "B"), ("X", "S", "B"), ("Y", "A", "S"), ("Z", "A", "Y")]),
    _g("three_and_pair", ["S", "X", "Y", "A", "B"], AB,
       [("S", "S", "S"), ("S", "A", "X"), ("S", "A", "B"), ("X", "S", "B"), ("Y", "A", "S")]),
    # scatters from two nonterminals
    _g("two_sources", ["S", "X", "Y", "Z", "A", "B"], AB,
       [("S", "A", "X"), ("X", "Y", "B"), ("Y", "A", "Z"), ("Z", "S", "B"), ("Z", "A", "B")]),
]


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
@pytest.mark.parametrize("n", [63, 128, 129, 256, 257, 450, 512])
def test_densities(cfpq, g, n):
    rng = np.random.default_rng(n)
    items = []
    for degree in (2, 5, 6, 8, 12, 24):
        for m in (degree * n, degree * n + 1):
            items.append((n, np.stack([rng.integers(0, n, m), rng.integers(0, 2, m), rng.integers(0, n, m)],
                                      axis=1).astype(np.int32), g))
    want = [worklist.closure(*it) for it in items]
    for it, w in zip(items, want):
        print("[gpu-case] resident density", g.name, n, len(it[1]), file=sys.stderr, flush=True)
        assert np.array_equal(cfpq.result_bits(cfpq.closure(*it)), w), len(it[1])
    print("[gpu-case] resident density, batch", g.name, n, file=sys.stderr, flush=True)
    for it, res, w in zip(items, cfpq.batch_closure(items), want):
        assert np.array_equal(cfpq.result_bits(res), w), len(it[1])
