"""Window statistics at the sizes where their kernels change form: the selection that holds 4, 8, 16
or 32 values per thread in one workgroup, then one workgroup per 4,096 values up to 128, from 2^22
values on 256; the EWMA
of one tile (up to 4,096 values) and of 2,048-value tiles, with last tiles of one to four values
and more tiles than the carry pass has threads. Quantiles bit for bit, the margin within one float32
ulp of the sequential EWMA and exactly the order statistic of the GPU's own values."""
import numpy as np
import pytest
import torch

import oracle
import paper_2606_12950_amd as M
from test_gpu_fitness import _t, gpu_quantiles

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("m", [4096, 4097, 8192, 8193, 16384, 16385, 32767, 36864, 36865, 524288, 524289, 600011,
                               2**22 - 1, 2**22, 2**22 + 5])
@pytest.mark.parametrize("kind", ["spread", "mixed", "equal"])
def test_quantiles_at_the_edges(m, kind):
    rng = np.random.default_rng(m)
    if kind == "spread":
        v = rng.standard_normal(m) * 10.0 ** rng.integers(-20, 20, m)
    else:
        v = np.where(rng.random(m) < 0.8, 0.0, rng.uniform(1, 500, m)) if kind == "mixed" else np.full(m, -2.5)
    v = v.astype(np.float32)
    print(f"quantiles m={m} {kind}", flush=True)
    for lo, hi in [(0.05, 0.95), (0.0, 1.0), (0.9, 0.9)]:
        assert gpu_quantiles(v, lo, hi).view(np.uint32).tolist() == oracle.quantiles(v, lo, hi).view(np.uint32).tolist()


@pytest.mark.parametrize("m", [4096, 4097, 4098, 4099, 4100, 6144, 6145, 8192, 2_099_199, 2_099_201, 2_101_250])
def test_margin_at_the_edges(m):
    rng = np.random.default_rng(m)
    pred = rng.uniform(1e9, 1e11, m)
    actual = pred * rng.lognormal(-0.05, 0.25, m)
    print(f"margin m={m}", flush=True)
    ew, rho = M.adaptive_rho(_t(actual), _t(pred), 0.2, 0.95)
    torch.cuda.synchronize()
    ew, rho = ew.cpu().numpy(), rho.cpu().numpy()
    want, _ = oracle.adaptive_rho(actual, pred, 0.2, 0.95)
    ulp = np.abs(ew.view(np.int32).astype(np.int64) - want.view(np.int32))
    assert ulp.max() <= 1 and (ulp == 0).mean() >= 0.999
    assert rho[0] == np.sort(ew)[int(np.ceil(0.95 * (m - 1)))]


def test_long_windows_use_the_whole_chip():
    # sixteen times the values: 5.6 times the time, 9.5 with 128 workgroups on 256 compute units
    def us(m):
        v, out = torch.randn(m, device="cuda"), torch.empty(2, device="cuda")
        ws = torch.empty(M._native.quantiles_workspace_bytes(m), dtype=torch.uint8, device="cuda")
        best = 1e9
        for _ in range(6):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(4):
                M.quantiles(v, out=out, workspace=ws)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 250)
        return best

    short, long = us(2**21), us(2**25)
    print(f"quantiles 2^21 {short:.1f} us, 2^25 {long:.1f} us", flush=True)
    assert long < 7.5 * short
