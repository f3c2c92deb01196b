"""The resident sweep (resident.h): the fixpoint of a small graph in one
workgroup, one, two and four lanes a row, at sizes around their edges; every
rule kind, products walked and multiplied by tiles, grammars it leaves to the
other resident kernel; single closures, a batch and max_iters, against the
oracle bit for bit."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import configs, graphs, grammars

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


SIZES = [1, 2, 31, 33, 64, 127, 128, 129, 255, 256, 257, 384, 385, 500, 512]


def _graph(n, degree, seed):
    return graphs.erdos_renyi(n, max(1, int(degree * n)), seed, labels=2)[1]


@pytest.mark.parametrize("g", GRAMMARS + [grammars.same_generation(), grammars.adjacent_layers()], ids=lambda g: g.name)
def test_resident_closures(cfpq, g):
    for n in SIZES:
        print("[gpu-case] resident", g.name, n, file=sys.stderr, flush=True)
        if g.terminals == grammars.HIERARCHY_TERMINALS:
            _, e = graphs.hierarchy(n, n, roots=max(1, n // 100), reverse=bool(n % 2))
        else:
            e = _graph(n, 1.5, 500 + n)
        want = worklist.closure(n, e, g)
        res = cfpq.closure(n, e, g)
        assert res.stats["converged"] == 1 and res.stats["path_used"] == 1
        assert np.array_equal(cfpq.result_bits(res), want), n
        assert not res.bits[:, n:].any()


@pytest.mark.parametrize("n", [96, 128, 200, 256, 300, 384, 450, 512])
@pytest.mark.parametrize("name", ["dyck", "transitive_closure", "same_generation", "anbn"])
def test_resident_dense(cfpq, n, name):
    """Dense closures: products by tiles from two lanes a row on."""
    g = grammars.BY_NAME[name]()
    if name == "same_generation":
        e = graphs.erdos_renyi_hier_labels(n, 4 * n, 7 + n)[1]
    else:
        e = _graph(n, 4, 7 + n)
    print("[gpu-case] resident dense", name, n, file=sys.stderr, flush=True)
    res = cfpq.closure(n, e, g)
    assert np.array_equal(cfpq.result_bits(res), worklist.closure(n, e, g))


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
def test_resident_one_lane_dense(cfpq, g):
    """One lane a row with transposed operands: from two edges a node on."""
    for n, degree in ((1, 2), (5, 3), (32, 2), (33, 4), (63, 6), (64, 2), (65, 3), (127, 5), (128, 2)):
        e = _graph(n, degree, 40 + n)
        print("[gpu-case] resident one lane", g.name, n, len(e), file=sys.stderr, flush=True)
        res = cfpq.closure(n, e, g)
        assert np.array_equal(cfpq.result_bits(res), worklist.closure(n, e, g)), n


def test_resident_batch_and_limits(cfpq):
    import torch
    items, want = [], []
    for q, n in enumerate(SIZES):
        g = GRAMMARS[q % len(GRAMMARS)]
        e = _graph(n, 2, 900 + n)
        items.append((n, torch.from_numpy(e).cuda() if q % 2 else e, g))
        want.append(worklist.closure(n, e, g))
    n, e = graphs.erdos_renyi(800, 2400, 3, labels=2)  # beside a large one
    items.append((n, e, grammars.dyck()))
    want.append(worklist.closure(n, e, grammars.dyck()))
    print("[gpu-case] resident batch", len(items), file=sys.stderr, flush=True)
    for use in (items, items[:-1], items[:-1][::-1]):
        res = cfpq.batch_closure(use)
        for (n, _, g), r in zip(use, res):
            i = [k for k, it in enumerate(items) if it[0] == n][0]
            assert np.array_equal(cfpq.result_bits(r), want[i]), (n, g.name)
    # a dense graph whose lists do not fit LDS, parallel edges, a cap, an edge out of range
    n = 500
    e = np.concatenate([graphs.erdos_renyi(n, 60000, 11, labels=2)[1]] * 2)
    res = cfpq.closure(n, e, grammars.anbn())
    assert np.array_equal(cfpq.result_bits(res), worklist.closure(n, e, grammars.anbn()))
    inst = configs.config1()
    full = worklist.closure(inst.n, inst.edges, inst.grammar)
    assert np.array_equal(cfpq.result_bits(cfpq.closure(inst.n, inst.edges, inst.grammar)), full)
    for cap in (1, 7, 1000):
        part = cfpq.closure(inst.n, inst.edges, inst.grammar, max_iters=cap, allow_partial=True)
        got = cfpq.result_bits(part)
        assert part.status == -4 and part.stats["iterations"] == cap
        assert got.any() and not (got & ~full).any()
    bad = inst.edges.copy()
    bad[3, 1] = 9
    with pytest.raises(cfpq.CfpqError) as ei:
        cfpq.closure(inst.n, torch.from_numpy(bad).cuda(), inst.grammar)
    assert ei.value.status == -1


@pytest.mark.parametrize("g", GRAMMARS, ids=lambda g: g.name)
def test_resident_follows_facts(cfpq, g):
    """Sparse graphs of one lane a row: chains and cycles (one or two bits a
    loop), hubs on both ends (lists past eight entries, many bits from one),
    and random trees, whose loops outgrow the facts one wavefront holds."""
    rng = np.random.default_rng(3)
    cases = []
    for n in (2, 33, 64, 128):
        chain = [(i, 0 if i < n // 2 else 1, i + 1) for i in range(n - 1)]
        cases.append((n, chain))
        cases.append((n, [(i, int(rng.integers(2)), int(rng.integers(n))) for i in range(n)]))
        cases.append((n, [(i, int(rng.integers(2)), (i + 1) % n) for i in range(n)]
                      + [(int(rng.integers(n)), int(rng.integers(2)), int(rng.integers(n))) for _ in range(n // 3)]))
    n = 100
    cases.append((n, [(0, 0, j) for j in range(1, 40)] + [(j, 1, 99) for j in range(1, 40)]
                  + [(99, 1, 50), (50, 1, 51), (51, 1, 52), (60, 0, 0), (61, 0, 60)]))
    for n, e in cases:
        e = np.asarray(e, np.int32)
        print("[gpu-case] resident facts", g.name, n, len(e), file=sys.stderr, flush=True)
        want = worklist.closure(n, e, g)
        res = cfpq.closure(n, e, g)
        assert np.array_equal(cfpq.result_bits(res), want), (n, len(e))
        assert res.stats["converged"] == 1
