"""The exact table where a block takes several radii and starts each from the
bracket of the one before (ascending, descending and shuffled radii, equal ones,
zero; a last group of fewer radii), at grids with a last block of few points, and
at the edge of the multipliers staged per block (1,024): W by bits, the lowest m
and the optimum against the oracle's scan over every multiplier."""
import numpy as np
import pytest

import oracle
from workloads.configs import Workload, _csr, _f32, eta_grid, lam_grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


def _check(ctx, dev, L, K, M, radii):
    import torch
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(K + M)
    parts = [rng.integers(0, L + 1, 300), rng.integers(1, 9, 50), np.full(7, L // 2)]
    C, E = len(parts), len(radii)
    off, xi = _csr([p.astype(np.int32) for p in parts])
    eps = np.repeat(np.asarray(radii, np.float64), C)
    w = Workload(f"radii-{E}", C, off, None, xi, np.full(C, L, np.int32), eta_grid(K, L),
                 lam_grid(M), _f32([10.0, 2.0, 0.5]), _f32([1.0, 1.0, 3.0]), E, _f32(eps))
    print(f"[gpu] table radii C={C} K={K} M={M} E={E}", flush=True)
    g = dro.dro_exact_table(ctx, dro.Problem.from_workload(w, dev), torch.from_numpy(w.eps).to(dev))
    torch.cuda.synchronize()
    ref = oracle.solve(w, grouped=True)
    for k in ("W", "W_star"):
        assert np.array_equal(g[k].cpu().numpy().view(np.uint64), ref[k].view(np.uint64)), k
    for k in ("m_star", "k_star", "m_at_star"):
        assert np.array_equal(g[k].cpu().numpy(), ref[k]), k


# 3 classes: 3 E / 4096 radii per block
@pytest.mark.parametrize("order", ["up", "down", "shuffled", "steps"])
@pytest.mark.parametrize("E,K,M", [(2731, 5, 17), (9001, 3, 40), (2800, 130, 9)])
def test_brackets_carry_over(ctx, dev, order, E, K, M):
    L = 200
    r = np.linspace(0.0, 0.6 * L, E)
    if order == "down":
        r = r[::-1].copy()
    if order == "shuffled":
        r = np.random.default_rng(E).permutation(r)
    if order == "steps":          # equal runs, back to zero now and then
        r = np.repeat(r[::7], 7)[:E]
        r[::97] = 0.0
    _check(ctx, dev, L, K, M, r)


@pytest.mark.parametrize("M", [1023, 1024, 1025])
@pytest.mark.parametrize("K", [127, 129])
def test_staged_multipliers(ctx, dev, M, K):
    _check(ctx, dev, 150, K, M, [3.0, 0.5, 20.0])
