"""Degradation plans (Alg. 2, Eq. 4) of nodes around one wavefront of engines: up to 64 engines sit
one per lane, more are ranked in strides. Steps and records bit for bit against the running sums
taken one engine after another in (level, index) order (numpy, same precision), with equal levels,
actions that free nothing or a negative amount, and neighbours of every size."""
import numpy as np
import pytest

from test_gpu_fitness import GB, gpu_plans

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("counts", [(63, 64, 65, 0, 1, 8, 9), (128, 129, 200, 64, 7), (1,), (64,), (65,)])
@pytest.mark.parametrize("levels", [5, 1])
def test_plans_around_a_wavefront(counts, levels):
    rng = np.random.default_rng(sum(counts) + levels)
    off = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    e = int(off[-1])
    level = rng.integers(6 - levels, 6, e).astype(np.int32)
    freed = rng.uniform(-5, 40, e) * GB
    freed[::7] = 0.0
    cost = rng.uniform(1, 5000, e).astype(np.float32)
    print(f"plans counts={counts} levels={levels}", flush=True)
    pf, pc, ne, raw, sf, sc, se = gpu_plans(off, level, freed, cost, 1500.0)
    assert ne.tolist() == list(counts)
    assert (raw[:, 100:104].copy().view(np.int32)[:, 0] == off[:-1]).all() and not raw[:, 104:].any()
    for j, n in enumerate(counts):
        f, top, c, hit = np.float64(0), None, np.float32(0), False
        for p, i in enumerate(sorted(range(off[j], off[j + 1]), key=lambda q: (level[q], q))):
            f, c, hit = f + freed[i], np.float32(c + cost[i]), hit or level[i] >= 4
            top = f if p == 0 else max(top, f)
            want = np.float32(c + np.float32(1500.0 if hit else 0.0))
            assert se[off[j] + p] == i and sf[off[j] + p] == top and sc[off[j] + p] == want, (j, p)
            if p < 8:
                assert pf[j, p] == top and pc[j, p] == want
        assert np.isposinf(pf[j, n:]).all() and (pc[j, n:] == 0).all()
