"""Single-path lengths where few new cells lie in many tiles and operands are
longer than 16, so that their min-plus walks single cells: chains with shuffled
node ids, whose lengths are the distances along the chain.  Steps of lengths up
to 16, up to 127 and beyond, with equal and different operands; one 4096-k pass,
a padded side that is no multiple of 1024, and a second pass."""
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


# S -> S S | a; S -> S T | a, T -> S S | a
GRAMMARS = {"same": SimpleNamespace(n_nonterminals=1, n_terminals=1, term=((0, 0),), bin=((0, 0, 0),)),
            "mixed": SimpleNamespace(n_nonterminals=2, n_terminals=1, term=((0, 0), (1, 0)),
                                     bin=((0, 0, 1), (1, 0, 0)))}


@pytest.mark.parametrize("rules", sorted(GRAMMARS))
@pytest.mark.parametrize("n", [1100, 2304, 4300])
def test_lengths_of_single_cells(cfpq, n, rules):
    print("[gpu-case] minplus cells", n, rules, file=sys.stderr, flush=True)
    g = GRAMMARS[rules]
    at = np.random.default_rng(n).permutation(n)  # position on the chain of every node
    node = np.argsort(at)
    e = np.stack([node[:-1], np.zeros(n - 1, np.int64), node[1:]], axis=1).astype(np.int32)
    _, got = cfpq.single_path(n, e, g)
    want = np.maximum(at[None, :] - at[:, None], 0).astype(np.uint32)
    for a in range(g.n_nonterminals):
        assert np.array_equal(got[a, :n, :n].cpu().numpy().view(np.uint32), want)
