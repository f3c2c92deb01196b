"""Row sweeps of graphs with nodes of thousands of edges, whose rows all
workgroups pull together: list lengths on both sides of where they do (512 k
words), one hub to more than the table holds, hubs that read each other, caps in
between -- against the dense products, and the oracle where it is fast."""
from __future__ import annotations

import sys

import numpy as np
import pytest

from oracle import worklist
from workloads import grammars, graphs

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


def _hubs(n, sizes, seed, extra):
    """Hubs with `sizes` outgoing edges (a, the next hub among their ends),
    half as many incoming ones (b), on random nodes, and `extra` random edges."""
    rng = np.random.default_rng(seed)
    node = rng.permutation(n)
    e = [graphs.erdos_renyi(n, extra, seed, labels=2)[1]]
    for q, size in enumerate(sizes):
        to = rng.choice(n, size=size, replace=False)
        to[0] = node[(q + 1) % len(sizes)]
        back = rng.choice(n, size=size // 2, replace=False)
        e.append(np.stack([np.full(size, node[q]), np.zeros(size, np.int64), to], axis=1))
        e.append(np.stack([back, np.ones(size // 2, np.int64), np.full(size // 2, node[q])], axis=1))
    return np.concatenate(e).astype(np.int32)


# hubs from 512 k words on: 16384 nodes 2048 entries, 8193 (132 words) 3971; none up to 8192
CASES = {"one": (16384, (16383,)), "edge": (16384, (2047, 2048, 2049)), "ring": (16384, (3000,) * 5),
         "too_many": (16384, (2060,) * 34), "wide": (8193, (3971, 3972, 8000)), "narrow": (4352, (3854, 3855, 4351)),
         "small": (4096, (4095, 4000))}


@pytest.mark.parametrize("case", sorted(CASES))
@pytest.mark.parametrize("g", [GRAMMARS[k] for k in (0, 1, 4, 5, 6)], ids=lambda g: g.name)
def test_hubs_equal_dense_products(cfpq, case, g):
    import torch
    n, sizes = CASES[case]
    d = torch.from_numpy(_hubs(n, sizes, 17, n // 4)).cuda()
    print("[gpu-case] sweep hubs", case, g.name, file=sys.stderr, flush=True)
    got = cfpq.closure(n, d, g, workspace=torch.full((1 << 30,), 1, dtype=torch.uint8, device="cuda"))
    want = cfpq.closure(n, d, g, path="fp4", hybrid=0)
    assert got.stats["converged"] == 1 and torch.equal(got.bits, want.bits)


@pytest.mark.parametrize("iters", [0, 1, 2, 3, 4])
def test_hubs_equal_oracle(cfpq, iters):
    n = 9000
    e = _hubs(n, (3700, 4500), 5, n // 8)
    for g in (grammars.anbn(), GRAMMARS[5]):
        want = worklist.closure(n, e, g)
        print("[gpu-case] sweep hubs, oracle", g.name, iters, file=sys.stderr, flush=True)
        res = cfpq.closure(n, e, g, max_iters=iters, allow_partial=True)
        got = cfpq.result_bits(res)
        assert not (got & ~want).any()
        assert (res.status == 0) == (res.stats["converged"] == 1)
        if res.status == 0:
            assert np.array_equal(got, want)
        else:
            assert iters > 0 and res.stats["iterations"] == iters
