"""Single-path lengths of a left-linear closure at the sizes where a row of
lengths fills 64 KiB of LDS (minplus_cols_row_kernel): complete layers of 256
nodes in chains of eight, so that a step has hundreds of new cells a row;
lengths are the differences of the layers."""
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


# on both sides of 64 KiB with and without the kernel's own 256 bytes, the largest, and one past it
@pytest.mark.parametrize("n", [16319, 16321, 16383, 16384, 16385])
def test_lengths_of_wide_rows(cfpq, n):
    import torch
    print("[gpu-case] minplus wide rows", n, file=sys.stderr, flush=True)
    layer = np.arange(n) // 256
    src = np.nonzero((layer % 8 < 7) & ((layer + 1) * 256 < n))[0]
    dst = (layer[src] + 1)[:, None] * 256 + np.arange(256)[None, :]
    e = np.stack([np.repeat(src, 256), np.zeros(dst.size, np.int64), dst.ravel()], axis=1)
    e = e[e[:, 2] < n].astype(np.int32)
    g = SimpleNamespace(n_nonterminals=2, n_terminals=1, term=((0, 0), (1, 0)), bin=((0, 0, 1),))  # S -> S A | a, A -> a
    _, got = cfpq.single_path(n, torch.from_numpy(e).cuda(), g)
    lay = torch.from_numpy(layer).cuda().to(torch.int32)
    want = torch.where(lay[None, :] // 8 == lay[:, None] // 8, lay[None, :] - lay[:, None], 0).clamp_(min=0)
    assert torch.equal(got[0, :n, :n], want)
    assert torch.equal(got[1, :n, :n], (want == 1).to(torch.int32))
    assert not got[:, n:].any() and not got[:, :, n:].any()
