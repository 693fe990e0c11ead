"""The small-batch predictor kernel against the large-batch one, bit for bit: a stage's prediction
takes the same sums in the same order in both, so the first n rows of a batch that the large-batch
kernel takes must come out the same when they are predicted as a batch of their own, for batch
sizes around the tiles of 64 (512-wide network) and 32 rows (1024-wide), the largest batch the
small-batch kernel takes and the first one beyond, and batches whose last rows it takes after whole
rounds of the large-batch kernel. Bins, two-phase heads and per-role regressors, with biases
that differ from neuron to neuron. (Both kernels are compared with the oracle elsewhere.)"""
import numpy as np
import pytest
import torch

import paper_2606_12950_amd as M

pytestmark = pytest.mark.gpu

NETS = {"mid": ((256, 512, 512, 64), 64, 256), "wide": ((256, 1024, 1024, 64), 32, 128)}


def _batch(net, n, seed, groups=None):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dims = NETS[net][0]
    lead = () if groups is None else (groups,)
    r = lambda *s: torch.randn(*s, generator=g, device="cuda")
    ws = [(r(*lead, o, i) * i ** -0.5).to(torch.bfloat16) for i, o in zip(dims[:-1], dims[1:])]
    bs = [r(*lead, o) * 0.3 for o in dims[1:]]
    x = r(n, dims[0]).to(torch.bfloat16)
    i = lambda hi: torch.randint(0, hi, (n,), generator=g, device="cuda", dtype=torch.int32)
    return dict(x=x, ws=ws, bs=bs, prompt=i(8000), model=i(9), role=i(6), tools=i(2),
                alpha=torch.rand(9, generator=g, device="cuda") * 1e5)


def _sizes(net):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    _, small, large = NETS[net]
    most, round_ = cus * small, cus * large
    return [1, small - 1, small, small + 1, 5 * small + 7, most - 1, most, most + 1, round_ + 1, round_ + small + 3,
            round_ + most, round_ + most + 1], round_ + large * 3 + round_ // 2


def _bins(b, n):
    c = 32.0 + 64.0 * torch.arange(64, device="cuda", dtype=torch.float32)
    return M.predict(b["x"][:n], b["ws"], b["bs"], c, b["prompt"][:n], b["model"][:n], b["alpha"])


def _heads(b, n):
    coef = torch.linspace(-2.5, 1.0, 64, device="cuda")
    knots = torch.linspace(0.0, 1.0, 9, device="cuda")
    head = torch.tensor([2, 3, 63, 1, 40], device="cuda", dtype=torch.int32)
    return M.predict_two_phase(b["x"][:n], b["ws"], b["bs"], head, coef, knots, knots * knots, 3000.0, b["prompt"][:n],
                               b["model"][:n], b["role"][:n], b["tools"][:n], b["alpha"])


@pytest.mark.parametrize("net", ["mid", "wide"])
@pytest.mark.parametrize("form", [_bins, _heads])
def test_small_batches_have_the_large_batch_bits(net, form):
    sizes, n = _sizes(net)
    b = _batch(net, n, 11)
    want = form(b, n)                        # its last half round is too long for the small-batch kernel
    for m in sizes:
        print(f"{net} {form.__name__} n={m}", flush=True)
        for got, ref in zip(form(b, m), want):
            assert torch.equal(got.view(torch.uint8), ref[:m].contiguous().view(torch.uint8)), m


@pytest.mark.parametrize("net", ["mid", "wide"])
@pytest.mark.parametrize("groups", [1, 3, 16])
def test_small_role_batches_have_the_large_batch_bits(net, groups):
    sizes, n = _sizes(net)
    b = _batch(net, n, 12)
    w = _batch(net, 1, 13, groups)
    reg = torch.tensor([0, groups - 1, groups // 2, -1, groups, 0], device="cuda", dtype=torch.int32)
    coef = torch.linspace(-2.0, 0.5, groups, device="cuda")
    p = torch.rand(n, device="cuda")

    def run(m):
        length, kv = torch.full((m,), -1.0, device="cuda"), torch.full((m,), -1.0, device="cuda", dtype=torch.float64)
        return M.predict_role_lengths(b["x"][:m], w["ws"], w["bs"], reg, coef, 1e5, b["prompt"][:m], b["model"][:m],
                                      b["role"][:m], p[:m], b["alpha"], length, kv)

    want = run(n)
    for m in sizes[:8]:
        print(f"{net} roles groups={groups} n={m}", flush=True)
        for got, ref in zip(run(m), want):
            assert torch.equal(got, ref[:m]), m
    b["role"].fill_(4 if groups == 1 else 3)   # no stage has a regressor: nothing is written
    assert (run(sizes[4])[0] == -1.0).all()


def _one_group_sizes():
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    small, half, full = 64 * cus, 128 * cus, 256 * cus
    return [small + 1, small + 129, half - 1, half, half + 1, full + small + 1, full + half, full + half + 1], 2 * full


@pytest.mark.parametrize("form", [_bins, _heads])
def test_one_row_group_has_the_bits_of_two(form):
    # the 512-wide network's 128-row tiles, for the rows past the last whole round of 256-row ones
    sizes, n = _one_group_sizes()
    b = _batch("mid", n, 14)
    want = form(b, n)
    for m in sizes:
        print(f"one group {form.__name__} n={m}", flush=True)
        for got, ref in zip(form(b, m), want):
            assert torch.equal(got.view(torch.uint8), ref[:m].contiguous().view(torch.uint8)), m


@pytest.mark.parametrize("groups", [1, 3, 16])
def test_one_row_group_role_tiles_have_the_bits_of_two(groups):
    sizes, n = _one_group_sizes()
    b = _batch("mid", n, 15)
    w = _batch("mid", 1, 16, groups)
    reg = torch.tensor([0, groups - 1, groups // 2, -1, 0, 0], device="cuda", dtype=torch.int32)
    coef = torch.linspace(-2.0, 0.5, groups, device="cuda")
    p = torch.rand(n, device="cuda")

    def run(m):
        length, kv = torch.full((m,), -1.0, device="cuda"), torch.full((m,), -1.0, device="cuda", dtype=torch.float64)
        return M.predict_role_lengths(b["x"][:m], w["ws"], w["bs"], reg, coef, 1e5, b["prompt"][:m], b["model"][:m],
                                      b["role"][:m], p[:m], b["alpha"], length, kv)

    want = run(n)
    for m in sizes[:5]:
        print(f"one group roles groups={groups} n={m}", flush=True)
        for got, ref in zip(run(m), want):
            assert torch.equal(got, ref[:m]), m
