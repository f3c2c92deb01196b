"""Single-path lengths on complete layers of 128 nodes: every k of a layer between
gives the same smallest sum, so that sums of powers of two meet their largest
values in each 128 k, at every length up to 32 (operands up to 16).  Lengths are
the differences of the layers."""
from __future__ import annotations

import sys
from types import SimpleNamespace

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


# the layers begin at a multiple of 128, or (skew) across the boundaries
@pytest.mark.parametrize("skew", [0, 40])
@pytest.mark.parametrize("layers", [21, 34])
def test_lengths_of_full_ties(cfpq, layers, skew):
    print("[gpu-case] minplus ties", layers, skew, file=sys.stderr, flush=True)
    n = 128 * layers + skew
    layer = np.full(n, -1)
    layer[skew:] = np.arange(128 * layers) // 128
    a = np.arange(skew, n - 128)
    src = np.repeat(a, 128)
    dst = (skew + 128 * (layer[a] + 1)[:, None] + np.arange(128)[None, :]).ravel()
    e = np.stack([src, np.zeros_like(src), dst], axis=1).astype(np.int32)
    g = SimpleNamespace(n_nonterminals=1, n_terminals=1, term=((0, 0),), bin=((0, 0, 0),))  # S -> S S | a
    _, got = cfpq.single_path(n, e, g)
    want = np.maximum(layer[None, :] - layer[:, None], 0).astype(np.uint32)
    want[:skew] = 0
    assert np.array_equal(got[0, :n, :n].cpu().numpy().view(np.uint32), want)
