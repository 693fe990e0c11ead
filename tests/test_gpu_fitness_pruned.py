"""Routing by fitness from bound tables (maestro_route_fitness_pruned, the form the binding takes
for large batches) against the kernel that scores every pair (maestro_route_fitness), which the
oracle checks cover: node indices and fitness bits identical, over every form both accept.

Node counts lie at the edges of the 64-node blocks, up to the largest the tables take. Ties are
forced by duplicated nodes, weights include classes outside [0, 1] and below 0 (where parts of the
bounds change side), headrooms include zero and negative ones, demands zero, none, far beyond
every node and (with a negative fit weight) negative ones, and ids out of range.
"""
import numpy as np
import pytest
import torch

import paper_2606_12950_amd as M
from paper_2606_12950_amd import _native, pipeline

pytestmark = pytest.mark.gpu

GB = 1.0e9
t = lambda a: pipeline._t(np.ascontiguousarray(a), "cuda")


def _inputs(seed, n, m, models, n_src, weights, free_gb, kv_gb, plans, tiers, deg_lo=0.0):
    rng = np.random.default_rng(seed)
    free = rng.uniform(0.0, free_gb, m)
    free[rng.random(m) < 0.02] = 0.0
    free[rng.random(m) < 0.01] = -1.0
    queue, act = rng.uniform(0, 5000, m).astype(np.float32), rng.uniform(2000, 20000, m).astype(np.float32)
    deg = np.where(rng.random(m) < 0.2, rng.uniform(1, 500, m), 0.0).astype(np.float32)
    rtt = rng.uniform(0.2, 80.0, (n_src, m)).astype(np.float32)
    mask = rng.integers(0, 2**63, m, dtype=np.int64)
    act_m = np.where(rng.random((m, models)) < 0.3, 0.0, rng.uniform(100, 20000, (m, models))).astype(np.float32)
    dup = rng.integers(0, m, m // 4)         # every fourth node is a copy of another: exact ties
    for a in (free, queue, act, deg, mask, act_m):
        a[:dup.size] = a[dup]
    rtt[:, :dup.size] = rtt[:, dup]
    kv = rng.uniform(0.0, kv_gb, n) * GB
    kv[::41] = 0.0
    kv[7::97] = 1e15
    model = rng.integers(0, models, n).astype(np.int32)
    src = rng.integers(0, n_src, n).astype(np.int32)
    cls = rng.integers(0, len(weights), n).astype(np.int32)
    model[11::53], src[12::53], cls[13::53] = models, -1, len(weights) + 3
    kw = dict(model_id=t(model), src_id=t(src), class_id=t(cls), kv_bytes=t(kv), free_bytes=t(free * GB),
              queue_ms=t(queue), act_ms=t(act), resident_mask=t(mask), deg_ms=t(deg), rtt_ms=t(rtt),
              class_weights=t(np.asarray(weights, np.float32)),
              bounds=t(np.array([0.5, 60.0, 300.0, 18000.0, deg_lo, 400.0], np.float32)), n_models=models)
    if tiers:
        kw.update(act_matrix=t(act_m), act_ms=None, resident_mask=None)
    if plans:
        count = np.where(rng.random(m) < 0.1, rng.integers(9, 30, m), rng.integers(0, 9, m))
        off = np.zeros(m + 1, np.int32)
        np.cumsum(count, out=off[1:])
        e = max(int(off[-1]), 1)
        kw["plans"] = M.degradation_plans(t(off), t(rng.integers(1, 6, e).astype(np.int32)[:off[-1]]),
                                          t(np.round(rng.uniform(0, 20, e))[:off[-1]] * GB),
                                          t(rng.uniform(0, 900, e).astype(np.float32)[:off[-1]]), 500.0)
    return kw


def _both(monkeypatch, **kw):
    lib = _native.load()
    used = []
    real = lib.maestro_route_fitness_pruned
    with monkeypatch.context() as mp:
        mp.setattr(lib, "maestro_route_fitness_pruned", lambda *a: (used.append(1), real(*a))[1])
        got = [a.cpu().numpy() for a in M.route_fitness(**kw)]
    assert used, "the sizes of this case must take the tables"
    with monkeypatch.context() as mp:
        mp.setattr(lib, "maestro_route_fitness_workspace", lambda *a: 0)
        want = [a.cpu().numpy() for a in M.route_fitness(**kw)]
    assert np.array_equal(got[0], want[0])
    assert np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32))
    return got


USUAL = [[0.25, 1, 1], [0.1, 1, 1]]
ODD = [[0.25, 1, 1], [1.5, 0.5, 2.0], [-0.3, 1, 0.0], [0.4, -0.7, 1.0], [0.2, 1.0, -0.8], [0.0, 0.0, 0.0]]


@pytest.mark.parametrize("m,models,k,n_src,free_gb,kv_gb,rho", [
    (64, 8, 1, 5, 288.0, 60.0, 0.0), (65, 33, 4, 1, 30.0, 10.0, 0.2), (127, 16, 2, 16, 30.0, 40.0, 0.0),
    (512, 16, 1, 5, 288.0, 2.0, 0.1), (1024, 8, 1, 2, 288.0, 4.0, 0.0), (1025, 8, 1, 3, 288.0, 0.5, 0.0),
    (1088, 5, 4, 2, 288.0, 1.0, 0.1), (1000, 64, 3, 5, 30.0, 3.0, 0.0), (2049, 7, 4, 3, 30.0, 25.0, 0.1),
    (4096, 64, 4, 5, 30.0, 2.0, 0.0), (4033, 1, 1, 2, 288.0, 2.0, 0.0)])
@pytest.mark.parametrize("plans", [False, True])
@pytest.mark.parametrize("tiers", [False, True])
def test_pruned_matches_every_pair(monkeypatch, m, models, k, n_src, free_gb, kv_gb, rho, plans, tiers):
    lib = _native.load()
    n = 1024
    while not lib.maestro_route_fitness_workspace(n, models, m, n_src, len(ODD), k, plans):
        n *= 2
    n += 333                                 # a ragged last workgroup, just past the size that takes the tables
    for weights, deg_lo in ((USUAL, 0.0), (ODD, -50.0)):
        print(f"pruned m={m} n={n} k={k} plans={plans} tiers={tiers} classes={len(weights)}", flush=True)
        kw = _inputs(m + k, n, m, models, n_src, weights, free_gb, kv_gb, plans, tiers, deg_lo)
        _both(monkeypatch, **kw, k=k, rho=rho)


def _takes_tables(kw, k):
    n, m = kw["kv_bytes"].shape[0], kw["free_bytes"].shape[0]
    need = M.route_fitness_workspace_bytes(n, kw["n_models"], m, kw["rtt_ms"].shape[0], kw["class_weights"].shape[0], k,
                                           "plans" in kw)
    ws = torch.full((max(need, 16),), 0xA5, dtype=torch.uint8, device="cuda")
    M.route_fitness(**kw, k=k, workspace=ws)
    return bool((ws != 0xA5).any())


# where the tables begin: from so many nodes on, from 2^pairs (stage, node) pairs on (0: any batch)
@pytest.mark.parametrize("k,plans,m,pairs", [
    (1, False, 2048, 0), (1, False, 256, 25), (1, False, 128, 26), (2, False, 3072, 0), (2, False, 192, 27),
    (3, False, 3072, 0), (3, False, 512, 27), (4, False, 512, 27), (1, True, 1024, 0), (1, True, 512, 24),
    (1, True, 192, 25), (1, True, 128, 26), (2, True, 1024, 0), (2, True, 640, 24), (2, True, 384, 25),
    (2, True, 192, 26), (3, True, 2000, 0), (4, True, 2000, 0), (3, True, 640, 25), (4, True, 384, 26)])
def test_where_the_tables_begin(monkeypatch, k, plans, m, pairs):
    n = -(-2 ** pairs // m) if pairs else 1025
    print(f"line k={k} plans={plans} m={m} n={n}", flush=True)
    below = _inputs(m, n, m - 1, 16, 5, ODD, 30.0, 10.0, plans, False)
    assert not _takes_tables(below, k)
    _both_routes(monkeypatch, **below, k=k)
    kw = _inputs(m + k, n, m, 16, 5, ODD, 30.0, 10.0, plans, m % 256 != 0, -50.0)
    assert _takes_tables(kw, k)
    _both_routes(monkeypatch, **kw, k=k)
    if pairs:
        kw = _inputs(m, n - 1, m, 16, 5, USUAL, 288.0, 60.0, plans, False)
        assert not _takes_tables(kw, k)
        _both_routes(monkeypatch, **kw, k=k)


def _both_routes(monkeypatch, **kw):
    got = [a.cpu().numpy().view(np.uint32) for a in M.route_fitness(**kw)]
    with monkeypatch.context() as mp:
        mp.setattr(_native.load(), "maestro_route_fitness_workspace", lambda *a: 0)
        want = [a.cpu().numpy().view(np.uint32) for a in M.route_fitness(**kw)]
    assert all(np.array_equal(a, b) for a, b in zip(got, want))


def test_pruned_without_admitting_nodes_and_with_negative_demand(monkeypatch):
    kw = _inputs(3, 70_001, 1100, 16, 5, ODD, 5.0, 1000.0, True, False)
    _both(monkeypatch, **kw, k=4)                 # nearly every pair short
    kw = _inputs(4, 70_001, 3100, 16, 5, ODD, 5.0, 1000.0, False, False)
    kw["free_bytes"].fill_(-1.0)
    _both(monkeypatch, **kw, k=2)                 # no node admits even an empty demand
    kw = _inputs(5, 70_001, 3100, 16, 5, ODD, 30.0, 10.0, False, False)
    kw["kv_bytes"].neg_()
    _both(monkeypatch, **kw, k=4)


@pytest.mark.parametrize("m,k,plans", [(600, 1, False), (600, 4, True), (2100, 4, False), (2100, 1, True)])
def test_pruned_with_headrooms_that_are_not_numbers(monkeypatch, m, k, plans):
    # such a node admits no stage (with plans it may free room), whatever the NaN's sign
    kw = _inputs(m + k, 140_003, m, 16, 5, USUAL, 30.0, 2.0, plans, False)
    kw["free_bytes"][3::29] = float("nan")
    kw["free_bytes"][5::31] = -float("nan")
    kw["kv_bytes"][::301] = float("nan")
    print(f"nan m={m} k={k} plans={plans}", flush=True)
    got = _both(monkeypatch, **kw, k=k)
    if not plans:
        nan = np.isnan(kw["free_bytes"].cpu().numpy())
        assert not nan[got[0][got[0] >= 0]].any() and (got[0][::301] == -1).all()


@pytest.mark.parametrize("m,k,plans", [(600, 1, False), (600, 4, True), (2100, 4, False), (2100, 1, True), (4096, 4, True)])
def test_pruned_where_penalties_overflow(monkeypatch, m, k, plans):
    # finite weights whose penalties pass the float32 range on some or all nodes: a pair that fits
    # and scores -inf is not listed, one that falls short is
    weights = [[0.25, 3e38, 3e38], [0.1, 2e38, 2.5e38], [0.25, 1.0, 1.0], [-0.3, 3.4e38, 3.4e38]]
    kw = _inputs(m + k, 140_003, m, 16, 5, weights, 30.0, 10.0, plans, False, -3000.0)
    kw["bounds"][2:4] = torch.tensor([-3000.0, 9000.0])
    print(f"overflow m={m} k={k} plans={plans}", flush=True)
    got = _both(monkeypatch, **kw, k=k)
    assert (got[0] == -1).any()


def test_pruned_on_a_stream_of_its_own(monkeypatch):
    kw = _inputs(6, 70_001, 3200, 16, 5, USUAL, 30.0, 2.0, False, False)
    want = _both(monkeypatch, **kw, k=4)
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    outs = [M.route_fitness(**kw, k=4, stream=s) for _ in range(3)]
    s.synchronize()
    for idx, fit in outs:
        assert np.array_equal(idx.cpu().numpy(), want[0])
        assert np.array_equal(fit.cpu().numpy().view(np.uint32), want[1].view(np.uint32))


def test_streams_that_are_not_torchs_and_capture_take_no_scratch(monkeypatch):
    kw = _inputs(7, 70_001, 3200, 16, 5, USUAL, 30.0, 2.0, False, False)
    want = _both(monkeypatch, **kw, k=4)
    torch.cuda.synchronize()

    class Handle:
        cuda_stream = torch.cuda.current_stream().cuda_stream

    lib = _native.load()
    out = (torch.empty(70_001, 4, dtype=torch.int32, device="cuda"), torch.empty(70_001, 4, device="cuda"))
    with monkeypatch.context() as mp:
        mp.setattr(lib, "maestro_route_fitness_pruned", None)      # not to be called
        M.route_fitness(**kw, k=4, out=out, stream=Handle())
        torch.cuda.synchronize()
        first = [a.cpu().numpy() for a in out]
        for a in out:
            a.zero_()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            M.route_fitness(**kw, k=4, out=out)
    for _ in range(3):
        graph.replay()
        torch.cuda.synchronize()
        for got in (first, [a.cpu().numpy() for a in out]):
            assert np.array_equal(got[0], want[0]) and np.array_equal(got[1].view(np.uint32), want[1].view(np.uint32))
        for a in out:
            a.zero_()


@pytest.mark.parametrize("plans", [False, True])
def test_workspace_of_the_caller(monkeypatch, plans):
    # nothing is allocated, and captured code and streams that are not torch's take the tables too
    n = 70_001
    kw = _inputs(8, n, 3200, 16, 5, USUAL, 30.0, 2.0, plans, False)
    want = _both(monkeypatch, **kw, k=4)
    out = (torch.empty(n, 4, dtype=torch.int32, device="cuda"), torch.empty(n, 4, device="cuda"))
    need = M.route_fitness_workspace_bytes(n, 16, 3200, 5, 2, 4, plans)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    lib, used = _native.load(), []
    real = lib.maestro_route_fitness_pruned
    monkeypatch.setattr(lib, "maestro_route_fitness_pruned", lambda *a: (used.append(a[-3]), real(*a))[1])

    def check(calls):
        torch.cuda.synchronize()
        assert used == [ws.data_ptr()] * calls
        for a, b in zip(out, want):
            assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))
            a.zero_()

    before = torch.cuda.memory_stats()["allocation.all.allocated"]
    M.route_fitness(**kw, k=4, out=out, workspace=ws)
    assert torch.cuda.memory_stats()["allocation.all.allocated"] == before
    check(1)

    class Handle:
        cuda_stream = torch.cuda.current_stream().cuda_stream

    M.route_fitness(**kw, k=4, out=out, workspace=ws, stream=Handle())
    check(2)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        M.route_fitness(**kw, k=4, out=out, workspace=ws)
    for _ in range(3):
        ws.random_(0, 255)                     # the program's own work between the replays
        graph.replay()
        check(3)
    with pytest.raises(_native.MaestroError, match="workspace"):
        M.route_fitness(**kw, k=4, out=out, workspace=ws[:need - 16])


def test_exhausted_memory_scores_every_pair(monkeypatch):
    kw = _inputs(9, 70_001, 3200, 16, 5, USUAL, 30.0, 2.0, False, False)
    want = _both(monkeypatch, **kw, k=1)

    def no_memory(*a):
        raise torch.OutOfMemoryError("no memory")

    monkeypatch.setattr(_native, "_scratch", no_memory)
    monkeypatch.setattr(_native.load(), "maestro_route_fitness_pruned", None)      # not to be called
    for a, b in zip(M.route_fitness(**kw, k=1), want):
        assert np.array_equal(a.cpu().numpy().view(np.uint32), b.view(np.uint32))


def test_pruned_argument_checks():
    lib = _native.load()
    assert lib.maestro_route_fitness_workspace(1000, 16, 512, 5, 2, 1, 0) == 0          # small batch
    assert lib.maestro_route_fitness_workspace(1 << 20, 16, 4097, 5, 2, 1, 0) == 0      # too many nodes
    assert lib.maestro_route_fitness_workspace(1 << 20, 16, 512, 5, 2, 5, 0) == 0       # long lists
    assert lib.maestro_route_fitness_workspace(1 << 20, 65, 512, 5, 2, 1, 0) == 0
    need = lib.maestro_route_fitness_workspace(1 << 20, 16, 512, 5, 2, 1, 0)
    assert need > 0
    p = torch.zeros(1 << 10, device="cuda").data_ptr()
    call = lambda n, ws, size: lib.maestro_route_fitness_pruned(
        n, p, p, p, p, 16, 512, 5, 2, p, p, p, p, None, p, None, None, p, p, p, 0.0, 1, p, p, ws, size, None)
    assert call(1 << 20, None, need) == 1
    assert call(1 << 20, p + 4, need) == 1
    assert call(1 << 20, p, need - 1) == 3
    assert call(1000, p, need) == 2
    assert call(-1, p, need) == 1
