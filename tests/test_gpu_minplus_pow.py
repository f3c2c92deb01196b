"""Single-path lengths at sizes where the min-plus of S -> S S runs on the
matrix cores (lengths as powers of two), ragged against its 128-cell tiles
and 64-k chunks, with equal and different operands, then on the VALU kernels
as the lengths grow: equal to the C oracle's."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import single_path as sp
from workloads import grammars, graphs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


# (n, edges, grammar): sparse random graphs; a graph above npad^2 / 16 edges
# (every rule a tile product, so operands differ); transitive closure (lengths
# past 16 beside short ones: a random part and a chain)
def _chain_and_random():
    n, e = graphs.erdos_renyi(1000, 2600, 21, labels=2)
    chain = np.array([[n + i, 0, n + i + 1] for i in range(99)], np.int32)
    return n + 100, np.concatenate([e, chain, np.array([[0, 0, n]], np.int32)]), grammars.transitive_closure()


CASES = {
    "er1030": lambda: (*graphs.erdos_renyi(1030, 4 * 1030, 22, labels=2), grammars.dyck()),
    "er1281": lambda: (*graphs.erdos_renyi(1281, 3 * 1281, 23, labels=2), grammars.dyck()),
    "dense1100": lambda: (*graphs.erdos_renyi(1100, 110000, 24, labels=2), grammars.dyck()),
    "chain_and_random": _chain_and_random,
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_lengths_on_matrix_cores(cfpq, name):
    n, e, g = CASES[name]()
    print("[gpu-case] minplus pow", name, n, len(e), file=sys.stderr, flush=True)
    want, loops, status = sp.lengths_native(n, e, g)
    assert status == 0
    res, got = cfpq.single_path(n, e, g)
    assert res.stats["iterations"] == loops and res.stats["minplus_terms"] > 0
    host = got[:, :n, :n].cpu().numpy().view(np.uint32)
    assert np.array_equal(host, want)
    assert not got[:, n:].any() and not got[:, :, n:].any()
