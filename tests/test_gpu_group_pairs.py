"""Batches of instances with several products a loop, at the sizes and densities
where they leave the group sweep for the tile engine: against the dense
products."""
from __future__ import annotations

import sys

import pytest

from workloads import graphs

from tests.test_gpu_sweep import GRAMMARS

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def cfpq():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1707_01007_amd as m
    m.lib()
    return m


def test_pairs_on_both_sides_of_the_line(cfpq):
    g = GRAMMARS[6]
    items = [(n, graphs.erdos_renyi(n, m, n + m, labels=2)[1], g)
             for n in (2048, 2049, 3000) for m in (n // 2, 2 * n, 2 * n + 1, 5 * n)]
    print("[gpu-case] group pairs", file=sys.stderr, flush=True)
    for (n, e, _), res in zip(items, cfpq.batch_closure(items)):
        assert bool((res.bits == cfpq.closure(n, e, g, path="fp4", hybrid=0).bits).all()), (n, len(e))
