"""The per-model node order (maestro_route_sort_nodes) where its buckets reach their limits: ready
times that are all equal, crowd just as many nodes into one bucket as it takes and one more, lie far
outside the others, differ in their last bits only, are signed zeros or not finite, at every launch
shape of the sort. Lists bit for bit against numpy's stable sort."""
import numpy as np
import pytest
import torch

import paper_2606_12950_amd as M
from test_gpu_route_split import _lists, _t

pytestmark = pytest.mark.gpu


def _key(f):
    u = f.view(np.uint32)
    return np.where(u >> 31, ~u, u | np.uint32(0x80000000))


@pytest.mark.parametrize("nodes", [1, 2, 63, 255, 256, 257, 512, 1000, 1024, 2047, 4096, 8191, 8192])
@pytest.mark.parametrize("kind", ["equal", "idle", "two", "most", "crowded", "outlier", "last_bits", "zeros", "infinite", "huge"])
def test_order_where_buckets_fill(nodes, kind):
    rng = np.random.default_rng(nodes)
    q = rng.uniform(0, 5, nodes).astype(np.float32)
    cold = np.zeros(nodes, np.float32)
    some = rng.permutation(nodes)
    if kind == "equal":
        q[:] = 2.5
    elif kind == "idle":                   # no queue; most nodes cold, by times of their own
        q[:] = 0.0
        cold = rng.uniform(2, 20, nodes).astype(np.float32)
    elif kind == "two":
        q[:] = 0.0
        cold[:] = 9.0
    elif kind in ("most", "crowded"):      # 32 equal ready times a bucket, or 33
        size = 32 if kind == "most" else 33
        q = np.sort(rng.uniform(1, 5, nodes)).astype(np.float32)
        q = np.repeat(np.arange((nodes + size - 1) // size, dtype=np.float32), size)[:nodes][some]
    elif kind == "outlier":
        q[some[0]] = 3e7
    elif kind == "last_bits":
        q = (np.float32(4.0).view(np.uint32) + rng.integers(0, 40, nodes).astype(np.uint32)).view(np.float32)
    elif kind == "zeros":
        q = np.where(rng.random(nodes) < 0.5, np.float32(-1e-30), np.float32(1e-30)).astype(np.float32)
        q[some[: nodes // 3]] = 0.0
        cold = np.where(rng.random(nodes) < 0.5, np.float32(-0.0), np.float32(0.0)).astype(np.float32)
        q[some[: nodes // 6]] = -0.0
    elif kind == "infinite":
        q[some[0]] = np.inf
    else:                                  # the span of the ready times overflows
        q[some[0]] = -3e38
        q[some[-1]] = 3e38
    mask = rng.integers(0, 4, nodes).astype(np.uint64)
    free = rng.uniform(0, 80e9, nodes)
    print(f"sort {kind} {nodes}", flush=True)
    got = _lists(M.route_sort_nodes(_t(free), _t(q), _t(cold), _t(mask), 3), 3, nodes)
    for m in range(3):
        res = ((mask >> np.uint64(m)) & np.uint64(1)) == 1
        ready = np.where(res, q + np.float32(0.0), q + cold).astype(np.float32)
        order = np.lexsort((np.arange(nodes), _key(ready)))
        assert np.array_equal(got[m]["node"], order.astype(np.int32))
        assert np.array_equal(got[m]["ready"].view(np.uint32), ready[order].view(np.uint32))
        assert np.array_equal(got[m]["free"], free[order])


def _check_order(nodes, q):
    free, mask = np.random.default_rng(nodes).uniform(0, 80e9, nodes), np.ones(nodes, np.uint64)
    got = _lists(M.route_sort_nodes(_t(free), _t(q), _t(np.zeros(nodes, np.float32)), _t(mask), 1), 1, nodes)
    assert np.array_equal(got[0]["node"], np.lexsort((np.arange(nodes), q)).astype(np.int32))


@pytest.mark.parametrize("nodes,most", [(255, 256), (256, 256), (512, 256), (600, 64), (1024, 64), (2048, 32), (4096, 32), (8192, 32)])
@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("spread", [False, True])
def test_order_at_the_bucket_limits(nodes, most, over, spread):
    # one bucket with as many equal ready times as it takes, or one more, among distinct ones; next to each
    # other (where the sample sees them) or spread over the nodes
    rng = np.random.default_rng(nodes + over)
    size = min(most + over, nodes - 2)
    q = rng.permutation(np.linspace(0, 9, nodes)).astype(np.float32)
    at = np.arange(nodes) if not spread else rng.permutation(nodes)
    q[at[:size]] = 4.5
    print(f"bucket limit nodes={nodes} size={size} spread={spread}", flush=True)
    _check_order(nodes, q)


def test_coarse_ready_times_are_not_sorted_twice():
    # 512 nodes, 8 queue lengths, residents or not: 1.3 times the time of distinct ready times, 1.6 where the
    # buckets gave up at 33 equal ones and radix passes followed
    rng = np.random.default_rng(5)
    nodes, models = 512, 8
    free, mask = _t(rng.uniform(0, 288e9, nodes)), _t(rng.integers(0, 2**63, nodes, dtype=np.int64) & rng.integers(
        0, 2**63, nodes, dtype=np.int64))
    lists = torch.empty(M._native.route_lists_bytes(models, nodes), dtype=torch.uint8, device="cuda")

    def us(q, cold):
        q, cold = _t(q.astype(np.float32)), _t(cold.astype(np.float32))
        run = lambda: M.route_sort_nodes(free, q, cold, mask, models, lists=lists)
        run()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            for _ in range(20):
                run()
        best = 1e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 50)
        return best

    fine = us(rng.uniform(0, 5, nodes), rng.uniform(2, 20, nodes))
    coarse = us(np.round(rng.uniform(0, 8, nodes)) * 0.5, np.full(nodes, 8.0))
    print(f"sort: distinct {fine:.2f} us, coarse {coarse:.2f} us", flush=True)
    assert coarse < 1.45 * fine
