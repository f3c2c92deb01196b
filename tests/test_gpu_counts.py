"""Bit-operations are counted for products of whole matrices only, on every
route: rules that a sweep applies and row gathers are sparse products."""
from __future__ import annotations

import sys

import pytest

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


SIZES = (40, 200, 500, 900, 3000)


def _check(cfpq, n, stats):
    dense = stats["products"] - stats["sparse_products"]
    assert 0 <= stats["sparse_products"] <= stats["products"] and stats["products"] > 0
    assert stats["bitops"] == 2.0 * cfpq.padded_rows(n) ** 3 * dense
    return dense


@pytest.mark.parametrize("name", ["anbn", "dyck"])
def test_only_dense_products_are_bit_operations(cfpq, name):
    g = grammars.BY_NAME[name]()
    items = [(n, graphs.erdos_renyi(n, 2 * n, n, labels=2)[1], g) for n in SIZES]
    print("[gpu-case] counts", name, file=sys.stderr, flush=True)
    with cfpq.Server(hbm_budget=1 << 30, hybrid_lanes=0) as srv:
        served = [srv.wait(srv.submit(*it))["stats"] for it in items]
    single = [cfpq.closure(*it).stats for it in items]
    batch = [r.stats for r in cfpq.batch_closure(items)]
    for n, *routes in zip(SIZES, single, batch, served):
        for st in routes:
            dense = _check(cfpq, n, st)
            if name == "anbn":  # every rule has an edge matrix
                assert dense == 0, n
            elif n > 512:       # S -> S S, once a loop at most
                assert 0 < dense <= st["iterations"], n
    # the kernels that multiply: every product on the resident one, the rules
    # without an edge matrix on the left on the tile engine
    for n, r in zip(SIZES, cfpq.batch_closure(items, dirty=False)):
        dense = _check(cfpq, n, r.stats)
        if n <= 512:
            assert r.stats["sparse_products"] == 0
        else:
            assert 0 < dense < r.stats["products"]
    for n, r in zip(SIZES, cfpq.batch_closure(items, hybrid=0)):
        if n > 512:
            assert _check(cfpq, n, r.stats) == r.stats["products"]
