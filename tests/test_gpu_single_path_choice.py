"""Single-path lengths around the least size whose tiles are worth another
kernel (768 nodes and one more), and where short rows are walked in place of the
matrix cores' powers of two (few edges a node): equal to the C oracle's."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import single_path as sp
from workloads import grammars, graphs

from tests.test_gpu_minplus_pow import cfpq  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,degree", [(20, 3), (768, 3), (769, 3), (769, 1), (1025, 1), (3000, 1)])
def test_lengths_around_the_choices(cfpq, n, degree):  # noqa: F811
    _, e = graphs.erdos_renyi(n, degree * n, 31, labels=1)
    g = grammars.transitive_closure()
    print("[gpu-case] single path choice", n, degree, file=sys.stderr, flush=True)
    want, loops, status = sp.lengths_native(n, e, g)
    assert status == 0
    res, got = cfpq.single_path(n, e, g)
    assert res.stats["iterations"] == loops
    host = got[:, :n, :n].cpu().numpy().view(np.uint32)
    assert np.array_equal(host, want)
