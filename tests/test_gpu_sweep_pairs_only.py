"""Grammars whose rules all join two growing nonterminals: the row sweeps up to
8192 nodes, the product loops, which work in place and take fewer loops, past
them."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from workloads import grammars

from tests.test_gpu_sweep import _g
from tests.test_gpu_workspace_routes import _bytes

pytestmark = pytest.mark.gpu

PAIRS = _g("pairs", ["S"], [("S", "a")], [("S", "S", "S")])
WITH_BASE = _g("base", ["S", "A"], [("S", "a"), ("A", "a")], [("S", "S", "S"), ("S", "A", "A")])
MIXED = _g("mixed", ["S", "A"], [("S", "a"), ("A", "a")], [("S", "S", "S"), ("S", "A", "S")])


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("n", [8192, 8193, 16384])
@pytest.mark.parametrize("g", [PAIRS, WITH_BASE, MIXED], ids=lambda g: g.name)
def test_chain_closure_and_route(cfpq, g, n):
    """A chain in random order: S reaches every later node.  One growing pair:
    the sweeps' matrices are part of the workspace exactly where the sweeps run."""
    at = np.random.default_rng(n).permutation(n)
    e = np.stack([at[:-1], np.zeros(n - 1, np.int64), at[1:]], 1).astype(np.int32)
    loops = _bytes(cfpq, n, e, g, profile=True)
    if g is PAIRS:
        assert (_bytes(cfpq, n, e, g) == loops) == (n > 8192)
    print("[gpu-case] pairs only", g.name, n, file=sys.stderr, flush=True)
    res = cfpq.closure(n, e, g)
    assert res.stats["converged"] == 1
    pos = np.empty(n, np.int64)
    pos[at] = np.arange(n)
    rng = np.random.default_rng(5)
    words = res.bits[0].cpu().numpy().view(np.uint64)
    for i in [int(at[0]), int(at[-1]), *map(int, rng.integers(0, n, 200))]:
        bits = np.unpackbits(words[i].view(np.uint8), bitorder="little")
        assert (bits[:n] == (pos > pos[i])).all() and not bits[n:].any()
