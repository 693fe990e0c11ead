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
