"""Loop caps that the product loops meet and the sweeps, which pass a fact from
rule to rule once a loop, would not: the closure converges as before.  And caps
that end both."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import grammars, graphs

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


# every rule reads what the one before it wrote: five sweeps, and one loop of
# products where these run one after another and one that changes nothing (513
# to 3840 nodes transpose the operands at a loop's start, so five and one)
STAIRS = _g("stairs", ["V", "W", "X", "Y", "Z", "A", "B"], [("A", "a"), ("B", "b")],
            [("Z", "A", "B"), ("Y", "A", "Z"), ("X", "B", "Y"), ("W", "A", "X"), ("V", "B", "W")])


@pytest.mark.parametrize("n,loops", [(40, 2), (100, 2), (200, 2), (500, 2), (513, 6), (1500, 6), (4200, 2)])
def test_cap_that_the_products_meet(cfpq, n, loops):
    _, e = graphs.erdos_renyi(n, 3 * n // 2, 70 + n, labels=2)
    want = worklist.closure(n, e, STAIRS)
    print("[gpu-case] cap met", n, file=sys.stderr, flush=True)
    res = cfpq.closure(n, e, STAIRS, max_iters=loops)
    assert res.stats["converged"] == 1 and res.stats["iterations"] <= loops
    assert np.array_equal(cfpq.result_bits(res), want)
    part = cfpq.closure(n, e, STAIRS, max_iters=1, allow_partial=True)
    assert part.status == -4 and part.stats["iterations"] == 1 and part.stats["converged"] == 0
    assert not (cfpq.result_bits(part) & ~want).any()
    res = cfpq.closure(n, e, STAIRS, max_iters=50)
    assert np.array_equal(cfpq.result_bits(res), want)


@pytest.mark.parametrize("cap", [1, 2, 3, 60])
def test_batch_of_capped_and_converged(cfpq, cap):
    items = []
    for n, g in ((60, STAIRS), (300, grammars.dyck()), (400, STAIRS), (600, grammars.anbn()), (700, STAIRS),
                 (64, grammars.transitive_closure()), (1100, STAIRS), (5000, STAIRS), (30, grammars.dyck())):
        items.append((n, graphs.erdos_renyi(n, 3 * n // 2, 11 + n, labels=2)[1], g))
    items.append((800, np.zeros((0, 3), np.int32), STAIRS))
    print("[gpu-case] batch cap", cap, file=sys.stderr, flush=True)
    done = 0
    for (n, e, g), res in zip(items, cfpq.batch_closure(items, max_iters=cap, allow_partial=True)):
        want, got = worklist.closure(n, e, g), cfpq.result_bits(res)
        assert not (got & ~want).any() and res.stats["iterations"] <= cap, n
        assert res.stats["converged"] == 0 or np.array_equal(got, want), n
        assert res.stats["converged"] == 1 or res.stats["iterations"] == cap, n
        assert not res.bits[:, n:].any()
        done += res.stats["converged"]
    assert done >= (len(items) if cap == 60 else 1)
    assert (res.status == 0) == (done == len(items))
