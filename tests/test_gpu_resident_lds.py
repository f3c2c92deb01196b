"""Small graphs whose adjacency lists fill the LDS: edge counts on both sides of
where a launch class's lists stop fitting and the graph goes to the other
resident kernel, alone, in a batch and in a server beside another request."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import grammars, graphs

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


# no rule with an edge matrix on the right and none over two growing operands:
# the kernel that may follow single facts, whatever the density
RIGHT = _g("right", ["S", "A"], [("S", "a"), ("A", "a")], [("S", "A", "S")])


def _edges(n, m):
    """Parallel edges included; few different ends, so that the closure is no
    full matrix."""
    rng = np.random.default_rng(m)
    return np.stack([rng.integers(0, n, m), np.zeros(m, np.int64), rng.integers(n // 2, n, m)], axis=1).astype(np.int32)


@pytest.mark.parametrize("n,counts", [
    (128, [19000, 19580, *range(19630, 19650, 3), 19700, 19834, 19835, 19866, 19896, 19897, 20100]),
    (127, [19590, 19650, 19860]), (129, list(range(19000, 20200, 200))), (300, list(range(17000, 19600, 200)))])
def test_lists_around_the_limit(cfpq, n, counts):
    items = [(n, _edges(n, m), RIGHT) for m in counts]
    want = [worklist.closure(*it) for it in items]
    for it, w in zip(items, want):
        print("[gpu-case] resident limit", n, len(it[1]), file=sys.stderr, flush=True)
        assert np.array_equal(cfpq.result_bits(cfpq.closure(*it)), w), len(it[1])
    print("[gpu-case] resident limit, batch", n, file=sys.stderr, flush=True)
    for it, res, w in zip(items, cfpq.batch_closure(items), want):
        assert np.array_equal(cfpq.result_bits(res), w), len(it[1])
    print("[gpu-case] resident limit, server", n, file=sys.stderr, flush=True)
    other = (200, graphs.erdos_renyi(200, 400, 8, labels=2)[1], grammars.dyck())
    with cfpq.Server(hbm_budget=1 << 30) as srv:
        tickets = [srv.submit(*it) for it in items + [other]]
        for it, t, w in zip(items + [other], tickets, want + [worklist.closure(*other)]):
            info = srv.wait(t)
            assert info["status"] == 0 and np.array_equal(cfpq.result_bits(info["result"]), w), len(it[1])


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
@pytest.mark.parametrize("n", [100, 200, 400])
def test_every_class_around_the_limit(cfpq, g, n):
    """Counts 12% apart over the range in which the lists stop fitting."""
    m = 4000
    while m < 45000:
        e = _edges(n, m)
        e[::3, 1] = 1
        print("[gpu-case] resident limit", g.name, n, m, file=sys.stderr, flush=True)
        assert np.array_equal(cfpq.result_bits(cfpq.closure(n, e, g)), worklist.closure(n, e, g)), m
        m += m // 8
