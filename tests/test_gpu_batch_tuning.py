"""The batch autotuner on sides whose instances run as group sweeps, where the
tile is no choice: one timing for both candidates and the route kept; a side
with an instance that the sweeps do not take is still tuned."""
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


def test_tiles_of_swept_sides_are_timed_once(cfpq):
    dense = graphs.erdos_renyi(1000, 17 * 1024, 3, labels=2)[1]  # more edges than the sweeps take
    items = [(n, graphs.erdos_renyi(n, 2 * n, n, labels=2)[1], grammars.dyck()) for n in (300, 600, 700, 900, 1200)]
    items.append((1000, dense, grammars.anbn()))
    cfpq.tune_clear()
    cfpq.batch_tune_set(768, "tiles", 128)
    print("[gpu-case] batch tuning", file=sys.stderr, flush=True)
    try:
        got = {e["npad"]: e for e in cfpq.batch_autotune(items, reps=3)}
        plain = {e["npad"]: e for e in cfpq.batch_autotune(items, reps=3, hybrid=0)}
    finally:
        cfpq.tune_clear()
    assert sorted(got) == sorted(plain) == [512, 768, 1024, 1280]
    for side in (768, 1280):
        c = got[side]["candidates_ms"]
        assert c["tiles256"] == c["tiles128"] == got[side]["ms"] > 0
        assert plain[side]["candidates_ms"]["tiles256"] != plain[side]["candidates_ms"]["tiles128"]
    assert got[768]["tile"] == 128 and got[1280]["tile"] == 256
    assert got[1024]["candidates_ms"]["tiles256"] != got[1024]["candidates_ms"]["tiles128"]
    assert len(set(got[512]["candidates_ms"].values())) == 3
