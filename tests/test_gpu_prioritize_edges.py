"""Slack ordering at the batch sizes where its launches change -- one workgroup up to 4,096 workflows
(one, two or four keys a thread; beyond 1,024 up to 32,768 stages), 1,024-key tiles up to 131,072, group
totals up to 1,024 tiles of 4,096 keys, group scans beyond -- bit for bit against the oracle: coarse deadlines (many equal keys,
so that stability shows), cursors anywhere, infinite latencies, and long chains among short ones."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_12950_amd as M
from paper_2606_12950_amd import pipeline

pytestmark = pytest.mark.gpu

t = lambda a: pipeline._t(np.ascontiguousarray(a), "cuda")


def _check(rng, lens, cursor=True, remaining=True, keys=50):
    W = len(lens)
    off = np.zeros(W + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    lat = rng.choice([0.5, 1.25, 3.0], int(off[-1])).astype(np.float32)
    lat[rng.random(lat.size) < 1e-3] = np.inf
    deadline = (rng.integers(0, keys, W) * 1_000_000).astype(np.int64)
    cur = rng.integers(-1, 9, W).astype(np.int32) if cursor else None
    print(f"prioritize W={W} S={lat.size} longest={max(lens)}", flush=True)
    rem, key, order = M.prioritize(t(off), t(lat), t(deadline), 7_000_000, cursor=None if cur is None else t(cur),
                                   want_remaining=remaining)
    torch.cuda.synchronize()
    want = oracle.prioritize(off, lat, deadline, 7_000_000, cursor=cur)
    assert np.array_equal(key.cpu().numpy(), want[1])
    assert np.array_equal(order.cpu().numpy(), want[2])
    if remaining:
        assert np.array_equal(rem.cpu().numpy(), want[0])


@pytest.mark.parametrize("W", [1, 63, 1023, 1024, 1025, 2047, 2048, 2049, 3071, 4095, 4096, 4097, 131072, 131073, 135168,
                               135169, 262145, 4194304, 4194305])
def test_orders_at_the_edges(W):
    rng = np.random.default_rng(W)
    _check(rng, rng.integers(0, 4, W), keys=50 if W < 10000 else 100000)


@pytest.mark.parametrize("W", [1, 1000, 1025, 4096])
@pytest.mark.parametrize("long_len", [1024, 1025, 2500, 9000])
def test_long_chains_in_one_workgroup(W, long_len):
    # ranges of a tile's stages within the staging capacity (short chains of none or one stage) and beyond; all of
    # one workgroup but 4,096 workflows of up to 11 stages and 9,000, whose 49,000 stages are tiled
    rng = np.random.default_rng(W + long_len)
    for hi in (2, 12):
        lens = rng.integers(0, hi, W)
        lens[rng.integers(0, W, 3)] = long_len
        _check(rng, lens, cursor=hi == 2, remaining=W != 1000)


@pytest.mark.parametrize("W", [1, 2, 64, 65, 300, 1024, 1025, 2049, 4096])
@pytest.mark.parametrize("kind", ["spread", "equal", "two", "most", "crowded", "saturated", "outlier"])
def test_one_workgroup_where_buckets_fill(W, kind):
    # keys that spread, that the buckets' special cases take, just fill a bucket, or overflow one
    rng = np.random.default_rng(W)
    lens = rng.integers(0, 4, W)
    off = np.zeros(W + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    lat = np.zeros(int(off[-1]), np.float32)         # the deadline alone sets the slack
    deadline = rng.integers(0, 2**31, W).astype(np.int64)
    if kind == "equal":
        deadline[:] = 123
    elif kind == "two":
        deadline = np.where(rng.random(W) < 0.5, 5, 9).astype(np.int64)
    elif kind in ("most", "crowded"):
        size = (64 if W <= 1024 else 32) + (kind == "crowded")    # bucket_most of one or several keys a thread
        deadline = rng.permutation(np.arange(W) // size * 1_000_000).astype(np.int64)
    elif kind == "saturated":
        deadline[rng.random(W) < 0.4] = 2**62
        deadline[rng.random(W) < 0.4] = -(2**62)
    elif kind == "outlier":
        deadline = rng.integers(0, 100_000, W).astype(np.int64)
        deadline[W // 2] = 2**62
    print(f"prioritize {kind} W={W}", flush=True)
    _, key, order = M.prioritize(t(off), t(lat), t(deadline), 1_000)
    torch.cuda.synchronize()
    want = oracle.prioritize(off, lat, deadline, 1_000)
    assert np.array_equal(key.cpu().numpy(), want[1]) and np.array_equal(order.cpu().numpy(), want[2])


@pytest.mark.parametrize("W,mean,one", [(1024, 8, True), (1024, 300, True), (1025, 31, True), (1025, 33, False), (2048, 15, True),
                                        (2048, 17, False), (4096, 7, True), (4096, 9, False), (4096, 100, False),
                                        (4096, 1100, False)])
def test_form_by_stages(W, mean, one):
    # one workgroup leaves the workspace as it is, the tiled launches keep keys and counts there
    rng = np.random.default_rng(W + mean)
    lens = rng.integers(mean - mean // 4, mean + mean // 4 + 1, W)
    off = np.zeros(W + 1, np.int64)
    np.cumsum(lens, out=off[1:])
    lat = rng.choice([0.5, 1.25, 3.0], int(off[-1])).astype(np.float32)
    deadline = rng.integers(0, 10**9, W).astype(np.int64)
    cur = rng.integers(-1, mean, W).astype(np.int32)
    ws = torch.full((M._native.prioritize_workspace_bytes(W, lat.size),), 0x5A, dtype=torch.uint8, device="cuda")
    print(f"prioritize W={W} S={lat.size}", flush=True)
    got = M.prioritize(t(off), t(lat), t(deadline), 7_000_000, cursor=t(cur), workspace=ws)
    torch.cuda.synchronize()
    assert bool((ws == 0x5A).all()) == one
    for a, b in zip(got, oracle.prioritize(off, lat, deadline, 7_000_000, cursor=cur)):
        assert np.array_equal(a.cpu().numpy(), b)
