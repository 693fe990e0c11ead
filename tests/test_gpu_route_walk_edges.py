"""The walk's block tables and the choice of algorithm at their edges: node counts around the blocks
of 8, 64 and 512 list entries, admitting nodes only at the edges of those blocks, demands of minus
infinity (every node admits, the blocks past the last node do not count) and of plus infinity, and
batches around the number of pairs from which the best node alone comes from the sorted lists.
Bars: node indices and score bits identical to the oracle's route and between the algorithms.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_12950_amd as M
from paper_2606_12950_amd import _native, pipeline

pytestmark = pytest.mark.gpu


def _t(a):
    return pipeline._t(np.ascontiguousarray(a), "cuda")


def _inputs(seed, n, nodes, models):
    rng = np.random.default_rng(seed)
    mask = rng.integers(0, 2 ** 63, nodes, dtype=np.int64).astype(np.uint64)
    return dict(model=rng.integers(0, models, n).astype(np.int32), pred=rng.uniform(32, 4064, n).astype(np.float32),
                kv=rng.choice(np.array([1.0, 3.0, 7.0]), n), dec=rng.uniform(0.01, 0.03, models).astype(np.float32),
                free=rng.uniform(0, 2, nodes), q=rng.choice(np.array([0.0, 0.5, 1.0, 2.0], np.float32), nodes),
                cold=rng.uniform(1, 20, nodes).astype(np.float32), mask=mask)


def _check(s, k, algos, sample=None):
    nodes, models = s["free"].shape[0], s["dec"].shape[0]
    rows = slice(None) if sample is None else sample
    ri, rs = oracle.route(s["model"][rows], s["pred"][rows], s["kv"][rows], s["dec"], s["free"], s["q"], s["cold"],
                          s["mask"], k=k, rho=0.0)
    args = [_t(s[name]) for name in ("model", "pred", "kv", "dec", "free", "q", "cold", "mask")]
    for algo in algos:
        gi, gs = M.route(*args, k=k, rho=0.0, algo=algo)
        torch.cuda.synchronize()
        gi, gs = gi.cpu().numpy()[rows], gs.cpu().numpy()[rows]
        assert np.array_equal(gi, ri), (nodes, models, k, algo)
        assert np.array_equal(gs.view(np.uint32), rs.view(np.uint32)), (nodes, models, k, algo)


@pytest.mark.parametrize("k", [1, 3, 16])
@pytest.mark.parametrize("nodes", [1, 7, 8, 9, 63, 64, 65, 511, 512, 513, 575, 1025, 4097, 8192])
def test_walk_at_block_edges(nodes, k):
    models = 3
    s = _inputs(nodes + k, 900, nodes, models)
    ready = np.where((s["mask"] & np.uint64(1)) == 1, s["q"], s["q"] + s["cold"])
    order = np.lexsort((np.arange(nodes), ready))          # model 0's list: headroom at its block edges
    edges = [j for j in (0, 7, 8, 15, 63, 64, 71, 127, 511, 512, 519, 1023, 1024, 4095, 4096, nodes - 1) if j < nodes]
    s["free"][order[edges]] = np.where(np.arange(len(edges)) % 3 == 0, 8.0, 4.0)
    s["kv"][::50] = -np.inf
    s["kv"][1::50] = np.inf
    _check(s, k, (M._native.ROUTE_SORTED, M._native.ROUTE_SCAN, M._native.ROUTE_AUTO))


@pytest.mark.parametrize("n,nodes,models", [(2 ** 17, 64, 8), (2 ** 17 + 1, 64, 8), (8191, 1024, 32), (8193, 1024, 32),
                                            (2048, 4096, 64), (2049, 4096, 64), (2 ** 23 + 1, 1, 1)])
def test_algorithm_choice_changes_no_result(n, nodes, models):
    s = _inputs(n, n, nodes, models)
    _check(s, 1, (M._native.ROUTE_AUTO,), sample=np.unique(np.r_[0:400, n // 2, n - 400:n]))


@pytest.mark.parametrize("n,nodes,models,lists", [
    (4096, 64, 8, False), (65_536, 64, 8, False), (4096, 64, 64, False), (1024, 512, 8, False),      # small products
    (131_073, 64, 8, True), (131_072, 64, 64, True), (1024, 512, 16, True), (16_384, 512, 8, True),
    (4096, 2048, 64, True), (1024, 8192, 64, True), (256, 8192, 8, True)])
def test_best_node_with_tiers_sorts_unless_the_scan_is_small(n, nodes, models, lists):
    # the scan leaves the workspace as it is, the sorted route writes its lists there
    s = _inputs(n, n, nodes, models)
    act = np.random.default_rng(n).uniform(0, 20, (nodes, models)).astype(np.float32)
    ws = torch.full((_native.route_workspace_bytes(n, models, nodes, 1),), 0x5A, dtype=torch.uint8, device="cuda")
    args = [_t(s[name]) for name in ("model", "pred", "kv", "dec", "free", "q")]
    print(f"tiers n={n} nodes={nodes} models={models}", flush=True)
    outs = []
    for algo, w in ((_native.ROUTE_AUTO, ws), (_native.ROUTE_SCAN, None), (_native.ROUTE_SORTED, None)):
        outs.append([a.cpu().numpy() for a in M.route(*args, None, None, k=1, rho=0.0, algo=algo, workspace=w,
                                                      act_s=_t(act))])
    assert bool((ws != 0x5A).any()) == lists
    for idx, score in outs[1:]:
        assert np.array_equal(outs[0][0], idx) and np.array_equal(outs[0][1].view(np.uint32), score.view(np.uint32))
