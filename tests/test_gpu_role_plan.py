"""The per-role regressors' bucketing where its plan changes place (in the scatter up to 1,024 blocks
of 1,024 stages, a launch of its own beyond) and at the edges of its blocks: a stage's length and KV
bytes do not depend on the other stages of the call, so every call must give the bits of calls over
sampled stages alone, and leave stages without a regressor as they were."""
import pytest
import torch

import paper_2606_12950_amd as M

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1023, 1024, 1025, 65537, 1 << 20, (1 << 20) + 1])
@pytest.mark.parametrize("groups", [1, 16])
def test_plan_in_place_and_apart(n, groups):
    g = torch.Generator(device="cuda")
    g.manual_seed(n + groups)
    r = lambda *s: torch.rand(*s, generator=g, device="cuda")
    ints = lambda hi: torch.randint(0, hi, (n,), generator=g, device="cuda", dtype=torch.int32)
    dims = (256, 512, 512, 64)
    ws = [(r(groups, o, i) - 0.5).mul_(2 * i ** -0.5).to(torch.bfloat16) for i, o in zip(dims[:-1], dims[1:])]
    bs = [r(groups, o) for o in dims[1:]]
    x = torch.empty(n, 256, device="cuda", dtype=torch.bfloat16)
    for i in range(0, n, 1 << 18):
        x[i:i + (1 << 18)] = r(min(1 << 18, n - i), 256).to(torch.bfloat16)
    role_regressor = torch.tensor([0, -1, groups - 1, groups, groups // 2], device="cuda", dtype=torch.int32)
    prompt, model, role, p = ints(8000), ints(7), ints(6), r(n)
    coef, alpha = r(groups), r(7) * 1e5
    print(f"roles n={n} groups={groups}", flush=True)

    def lengths(rows):
        out = torch.full((rows.numel(),), -1.0, device="cuda"), torch.full((rows.numel(),), -2.0, device="cuda",
                                                                            dtype=torch.float64)
        return M.predict_role_lengths(x[rows], ws, bs, role_regressor, coef, 32768.0, prompt[rows], model[rows],
                                      role[rows], p[rows], alpha, *out)

    got = lengths(torch.arange(n, device="cuda"))
    for size in (1, 700):
        rows = torch.unique(torch.cat([torch.randint(0, n, (size,), generator=g, device="cuda"),
                                       torch.tensor([0, n - 1], device="cuda")]))
        want = lengths(rows)
        assert torch.equal(got[0][rows], want[0]) and torch.equal(got[1][rows], want[1])
    own = (role == 0) | (role == 2) | (role == 4)
    assert bool((got[0][~own] == -1.0).all()) and bool((got[1][~own] == -2.0).all())
    assert bool((got[0][own] >= 0.0).all()) and bool((got[1][own] >= 0.0).all())
