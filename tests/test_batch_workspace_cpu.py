"""Workspace of batches of small instances (host only): instances in a row share
their grammar's table, by its content, and no part of a batch needs more than
the whole."""
from __future__ import annotations

import ctypes
import os
from types import SimpleNamespace

import numpy as np
import pytest

from workloads import grammars


def _bytes(cfpq, items, copies=False):
    from paper_1707_01007_amd import _abi
    rec = (_abi.Instance * len(items))()
    keep = []
    for i, (n, m, g) in enumerate(items):
        gs, kg = cfpq._grammar_struct_new(g) if copies else cfpq._grammar_struct(g)
        e = np.zeros((m, 3), np.int32)
        keep += [gs, kg, e]
        rec[i] = _abi.Instance(_abi.Graph(n, 0, m, ctypes.c_void_p(e.ctypes.data)), ctypes.pointer(gs),
                               ctypes.c_void_p(1 << 20))
    size = ctypes.c_size_t(0)
    _abi.check(cfpq.lib().cfpq_batch_workspace_bytes(len(items), rec, None, ctypes.byref(size)))
    return size.value


@pytest.fixture(scope="module")
def cfpq():
    import paper_1707_01007_amd as m
    from paper_1707_01007_amd import _abi
    if not os.path.exists(_abi.LIB_PATH):
        pytest.skip("libcfpq.so not built")
    return m


# 21 binary rules: beyond the resident sweep's tables
MANY = SimpleNamespace(n_nonterminals=6, n_terminals=1, term=((0, 0),),
                       bin=tuple((i % 6, (i + 1) % 6, (i + 2 + i // 6) % 6) for i in range(21)))


def test_sizes_follow_the_grammars_content(cfpq):
    gs = [grammars.dyck(), grammars.anbn(), grammars.same_generation(), MANY]
    rng = np.random.default_rng(2)
    items = [(int(n), int(n * d), gs[int(k)]) for n, d, k in
             zip(rng.integers(1, 700, 60), rng.integers(0, 5, 60), rng.integers(0, 4, 60))]
    whole = _bytes(cfpq, items)
    assert whole == _bytes(cfpq, items, copies=True)
    for _ in range(20):
        part = [items[i] for i in sorted(rng.choice(60, size=int(rng.integers(1, 60)), replace=False))]
        assert 0 < _bytes(cfpq, part) <= whole


def test_one_grammar_is_kept_once(cfpq):
    g = grammars.anbn()
    assert _bytes(cfpq, [(30, 20, g), (30, 90, g)] * 500) > _bytes(cfpq, [(30, 20, g)] * 500 + [(30, 90, g)] * 500)
