"""Fitness routing from bound tables where bounds prune little. Nodes that tie: clusters of idle nodes of one kind, whose scores
differ by the source's round-trip time, by residency or by nothing, so that the block bounds of most nodes
reach the best score. And with plans, nodes that all fall short: without headroom, of one headroom, with
plans that never free enough. Node indices and fitness bits against scoring every pair, and the time:
visiting every tie, and every short pair by one wavefront, took three to ten times as long as scoring
every pair."""
import numpy as np
import pytest
import torch

import paper_2606_12950_amd as M
from paper_2606_12950_amd import _native
from test_gpu_fitness_pruned import ODD, USUAL, _both, _inputs, _takes_tables

pytestmark = pytest.mark.gpu

GB = 1.0e9


def _idle(kw, kind):
    m = kw["free_bytes"].shape[0]
    kw["free_bytes"].fill_(200 * GB)
    kw["queue_ms"].zero_()
    if kw["deg_ms"] is not None:
        kw["deg_ms"].zero_()
    region = torch.arange(m, device="cuda") % (4 if kind != "one" else 1)
    kw["rtt_ms"].copy_(kw["rtt_ms"][:, :4][:, region])
    if kw["resident_mask"] is not None:
        if kind == "one":
            kw["resident_mask"].fill_(-1)
        kw["act_ms"].fill_(8000.0)
    if kind == "steps":                      # headrooms and queues of a few distinct values
        kw["free_bytes"].copy_(torch.where(region < 2, 200 * GB, 150 * GB))
        kw["queue_ms"].copy_((torch.arange(m, device="cuda") * 7 % 3).float() * 2000)
    return kw


@pytest.mark.parametrize("n,m,k", [(2**19, 128, 1), (2**16, 512, 1), (2**18, 512, 4), (134_300, 1000, 3),
                                   (122_100, 1100, 2), (2**16, 2049, 4), (1024, 4096, 1), (1024, 4096, 4)])
@pytest.mark.parametrize("kind", ["one", "regions", "steps"])
@pytest.mark.parametrize("plans", [False, True])
def test_ties_match_every_pair(monkeypatch, n, m, k, kind, plans):
    print(f"ties m={m} n={n} k={k} {kind} plans={plans}", flush=True)
    for weights, tiers in ((USUAL, False), (ODD, m == 512)):
        kw = _idle(_inputs(m + k, n + 77, m, 16, 5, weights, 30.0, 10.0, plans, tiers), kind)
        assert _takes_tables(kw, k)
        _both(monkeypatch, **kw, k=k)


def _saturated(kw, kind):
    m = kw["free_bytes"].shape[0]
    kw["free_bytes"].fill_(0.0 if kind != "same" else 1e6)
    kw["kv_bytes"].clamp_(min=2e6)
    off = torch.arange(m + 1, device="cuda", dtype=torch.int32) * 3
    e = 3 * m
    r = torch.Generator(device="cuda").manual_seed(m)
    level = torch.randint(1, 6, (e,), generator=r, device="cuda", dtype=torch.int32)
    freed = torch.rand(e, generator=r, device="cuda", dtype=torch.float64) * (0.1 if kind == "fail" else 20) * GB
    cost = torch.rand(e, generator=r, device="cuda") * 900
    if kind == "mixed":
        kw["kv_bytes"][torch.arange(kw["kv_bytes"].shape[0], device="cuda") // 64 % 3 == 0] = 0.0
        kw["free_bytes"][::5] = 1e6 * torch.rand(m, generator=torch.Generator(device="cuda").manual_seed(m),
                                                 device="cuda", dtype=torch.float64)[::5]
    if kind == "same":
        kw = _idle(kw, "regions")
        kw["free_bytes"].fill_(1e6)
        level.fill_(1), freed.fill_(20 * GB), cost.fill_(300.0)
    if kind == "long":                       # 0 .. 40 engines, most past a plan's record
        off[1:] = torch.cumsum(torch.randint(0, 41, (m,), generator=r, device="cuda"), 0)
        e = int(off[-1])
        level = torch.randint(1, 6, (e,), generator=r, device="cuda", dtype=torch.int32)
        freed = torch.rand(e, generator=r, device="cuda", dtype=torch.float64) * GB
        cost = torch.rand(e, generator=r, device="cuda") * 90
    if kind == "none":
        off.zero_()
        level, freed, cost = level[:0], freed[:0], cost[:0]
    kw["plans"] = M.degradation_plans(off, level, freed, cost, 500.0)
    return kw


@pytest.mark.parametrize("n,m,k", [(4_000, 2_049, 4), (8_192, 4_096, 1), (30_001, 2_049, 3), (50_001, 2_049, 2), (100_003, 1_100, 1),
                                   (70_000, 1_024, 4), (300_001, 600, 3)])
@pytest.mark.parametrize("kind", ["empty", "same", "fail", "none", "mixed", "long"])
def test_short_of_room_everywhere_matches_every_pair(monkeypatch, n, m, k, kind):
    # 8, 4, 2 and 1 wavefronts that share the short pairs of 64 stages; ragged last groups; "mixed": two groups
    # of 64 stages in three short of room on every node, with headrooms that differ
    print(f"saturated m={m} n={n} k={k} {kind}", flush=True)
    for weights in (USUAL, ODD):
        kw = _saturated(_inputs(m + k, n, m, 16, 5, weights, 30.0, 10.0, True, False), kind)
        assert _takes_tables(kw, k)
        got = _both(monkeypatch, **kw, k=k)
        assert (got[0][:, 0] == -1).all() == (kind == "none")


def _us(f):
    f()
    best = 1e9
    for _ in range(5):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(4):
            f()
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 250)
    return best


@pytest.mark.parametrize("n,m,k,kind", [(719_712, 512, 1, "one"), (719_712, 512, 1, "regions"), (131_072, 4096, 4, "regions"),
                                        (4096, 4096, 1, "one")])
def test_ties_take_no_longer_than_every_pair(monkeypatch, n, m, k, kind):
    # measured 0.4 .. 0.7 of that time; 3 to 10 times it with every tie visited
    _time(monkeypatch, _idle(_inputs(m, n, m, 16, 5, USUAL, 30.0, 2.0, False, False), kind), n, m, k, kind)


@pytest.mark.parametrize("n,m,k,kind", [(8192, 4096, 1, "same"), (8192, 4096, 1, "empty"), (32_768, 4096, 4, "fail")])
def test_short_of_room_takes_no_longer_than_every_pair(monkeypatch, n, m, k, kind):
    # measured 0.7 .. 1.05 of that time; 3 to 9 times it with one wavefront for the short pairs of 64 stages
    _time(monkeypatch, _saturated(_inputs(m, n, m, 16, 5, USUAL, 30.0, 10.0, True, False), kind), n, m, k, kind)


def _time(monkeypatch, kw, n, m, k, kind):
    out = (torch.empty(n, k, dtype=torch.int32, device="cuda"), torch.empty(n, k, device="cuda"))
    lib = _native.load()
    assert _takes_tables(kw, k)
    tables = _us(lambda: M.route_fitness(**kw, k=k, out=out))
    monkeypatch.setattr(lib, "maestro_route_fitness_workspace", lambda *a: 0)
    every = _us(lambda: M.route_fitness(**kw, k=k, out=out))
    print(f"bounds n={n} m={m} k={k} {kind}: tables {tables:.1f} us, every pair {every:.1f} us", flush=True)
    assert tables < 1.5 * every
