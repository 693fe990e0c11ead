"""Scratch that the binding takes for a call belongs to the stream that runs the call: taken from the
current stream's pool instead, its block would be given to that stream's next tensor while the other
stream still works in it. On the CPU with the library, the streams and the allocator replaced by
recorders; on the GPU by address (the streams idle between the steps)."""
import contextlib
import types

import pytest
import torch

import paper_2606_12950_amd as M
from paper_2606_12950_amd import _native

i32, f32, f64, i64 = torch.int32, torch.float32, torch.float64, torch.int64


def _calls(dev):
    """Every call that takes scratch of its own, without a workspace, its inputs and outputs at hand."""
    n, m, k, w, win = 64, 16, 4, 32, 40_000
    z = lambda *s, dtype=f32: torch.zeros(*s, dtype=dtype, device=dev)
    dims = (256, 512, 512, 64)
    ws = [z(1, o, i, dtype=torch.bfloat16) for i, o in zip(dims[:-1], dims[1:])]
    bs = [z(1, o) for o in dims[1:]]
    off = torch.arange(w + 1, dtype=i64, device=dev)
    ids, rows, kv, per_model = z(n, dtype=i32), z(n), z(n, dtype=f64), z(k)
    node = (z(m, dtype=f64) + 1, z(m), z(m), z(m, dtype=i64))
    routed = (z(n, 2, dtype=i32), z(n, 2))
    x, role, one, pred, kv_out = z(n, 256, dtype=torch.bfloat16), z(1, dtype=i32), z(1), z(n), z(n, dtype=f64)
    values, bounds, ratio, ewma, rho = z(win), z(2), z(win, dtype=f64) + 1, z(win), z(1)
    latency, deadline, ordered = z(w), z(w, dtype=i64), (z(w, dtype=i64), z(w, dtype=i32), z(w, dtype=i32))
    return {
        "maestro_route_ex": lambda s: M.route(ids, rows, kv, per_model, *node, k=2, out=routed, stream=s),
        "maestro_predict_role_lengths": lambda s: M.predict_role_lengths(
            x, ws, bs, role, one, 100.0, ids, ids, ids, rows, per_model, pred, kv_out, stream=s),
        "maestro_quantiles": lambda s: M.quantiles(values, out=bounds, stream=s),
        "maestro_adaptive_rho": lambda s: M.adaptive_rho(ratio, ratio, 0.2, 0.9, out=(ewma, rho), stream=s),
        "maestro_prioritize": lambda s: M.prioritize(off, latency, deadline, 0, out=ordered, stream=s),
    }


CALLS = sorted(_calls("cpu"))


@pytest.mark.parametrize("name", CALLS)
@pytest.mark.parametrize("kind", ["torch", "handle"])
def test_scratch_is_taken_under_the_launch_stream(monkeypatch, name, kind):
    class Stream:                             # stands for torch.cuda.Stream
        cuda_stream = 4096

    class External(Stream):
        def __init__(self, handle, device=None):
            self.cuda_stream = handle

    current, taken, launched = [None], [], []

    @contextlib.contextmanager
    def on(s):
        old, current[0] = current[0], s.cuda_stream
        yield
        current[0] = old

    real_empty = torch.empty

    def empty(*a, **kw):
        if kw.get("dtype") == torch.uint8:
            taken.append(current[0])
        return real_empty(*a, **kw)

    call = _calls("cpu")[name]
    lib = types.SimpleNamespace(**{f: (lambda *a: 4096) for f in (
        "maestro_route_workspace", "maestro_role_lengths_workspace", "maestro_quantiles_workspace",
        "maestro_prioritize_workspace")})
    setattr(lib, name, lambda *a: (launched.append(a), 0)[1])
    monkeypatch.setattr(_native, "load", lambda: lib)
    monkeypatch.setattr(_native, "_dev", lambda t, *a: t)
    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "ExternalStream", External)
    monkeypatch.setattr(torch.cuda, "stream", on)
    monkeypatch.setattr(torch, "empty", empty)
    handle = Stream() if kind == "torch" else types.SimpleNamespace(cuda_stream=8192)
    call(handle)
    assert taken == [handle.cuda_stream]
    assert launched[0][-1] == handle.cuda_stream


@pytest.mark.parametrize("capturing", ["neither", "current", "launch"])
def test_no_scratch_while_a_stream_is_captured(monkeypatch, capturing):
    # a call on another stream, itself not captured, still allocates in the capturing thread
    class Stream:
        pass

    current = [None]

    @contextlib.contextmanager
    def on(s):
        old, current[0] = current[0], s
        yield
        current[0] = old

    launch = Stream()
    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "stream", on)
    captured = {"neither": "no stream", "current": None, "launch": launch}[capturing]
    monkeypatch.setattr(torch.cuda, "is_current_stream_capturing", lambda: current[0] is captured)
    assert _native._may_allocate(launch) == (capturing == "neither")
    assert _native._may_allocate(None) == (capturing != "current")
    assert not _native._may_allocate(types.SimpleNamespace(cuda_stream=1))


@pytest.mark.gpu
@pytest.mark.parametrize("name", CALLS)
def test_current_stream_is_not_given_the_block(monkeypatch, name):
    lib, used = _native.load(), []            # address and size of each call's scratch
    call = _calls("cuda")[name]
    side = torch.cuda.Stream()
    handle = types.SimpleNamespace(cuda_stream=side.cuda_stream)
    real = getattr(lib, name)

    def record(*a):
        used.append(a[-3:-1])                 # the arguments before the stream
        return real(*a)

    monkeypatch.setattr(lib, name, record)
    for s in (side, handle):
        torch.cuda.synchronize()
        print(f"scratch {name} {type(s).__name__}", flush=True)
        call(s)
        torch.cuda.synchronize()
        address, size = used[-1]
        assert address not in {torch.empty(size, dtype=torch.uint8, device="cuda").data_ptr() for _ in range(4)}
    assert used[0] == used[1]                 # one stream, by either name: one pool


@pytest.mark.parametrize("missing", [(), ("_cuda_getDevice",), ("_cuda_getCurrentRawStream",)])
def test_current_stream_without_torchs_private_calls(monkeypatch, missing):
    class Torch:                              # torch with some of its private calls gone
        class cuda:
            current_stream = staticmethod(lambda: types.SimpleNamespace(cuda_stream=4096))

        class _C:
            _cuda_getDevice = staticmethod(lambda: 3)
            _cuda_getCurrentRawStream = staticmethod(lambda device: 4096 if device == 3 else 0)

    for name in missing:
        delattr(Torch._C, name)
    monkeypatch.setattr(_native, "torch", Torch)
    assert _native._stream(None) == 4096
    assert _native._stream(types.SimpleNamespace(cuda_stream=64)) == 64
