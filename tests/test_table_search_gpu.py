"""The exact table's search over the multipliers where its shortcuts end, against
the oracle's scan over every multiplier (W by bits, the lowest m, the optimum):
one and two multipliers, grids past the block's staged ones (1,024), radii at
which J is flat or nearly flat in the multiplier (every sample at the radius, so
that the slope is zero over many multipliers; radius 0; radii a rounding away),
and multipliers above and below both costs.  A multiplier grid that is not
ascending is outside the contract and is scanned: compared with the oracle on
the same order.
"""
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


def _check(ctx, dev, w):
    import torch
    import paper_2607_16892_amd as dro
    print(f"[gpu] table search {w.name}: C={w.C} K={w.K} M={w.M} E={w.E}", flush=True)
    prob = dro.Problem.from_workload(w, dev)
    g = dro.dro_exact_table(ctx, prob, torch.from_numpy(w.eps).to(dev))
    torch.cuda.synchronize()
    ref = oracle.solve(w, grouped=True)
    for k in ("W", "W_star"):
        assert np.array_equal(g[k].cpu().numpy().view(np.uint64), ref[k].view(np.uint64)), k
    for k in ("m_star", "k_star", "m_at_star"):
        assert np.array_equal(g[k].cpu().numpy(), ref[k]), k


def _workload(name, L, K, lam, E):
    rng = np.random.default_rng(len(lam) + K)
    parts = [np.full(1, 10), np.full(37, 10), np.full(5, 0), np.full(5, L),
             rng.integers(0, L + 1, 400), np.array([3, 17, 10, 10])]
    C = len(parts)
    off, xi = _csr([p.astype(np.int32) for p in parts])
    c_p = _f32([8.0, 1.0, 0.5, 3.0, 40.0, 2.0 ** 7])
    c_w = _f32([1.0, 1.0, 3.0, 3.0, 0.25, 2.0 ** -10])
    base = np.array([0.0, 10.0, np.nextafter(np.float32(10), np.float32(11)), 1e-7, L / 2.0, 9.75,
                     1e-3 * L, float(L)][:E])
    return Workload(name, C, off, None, xi, np.full(C, L, np.int32), eta_grid(K, L), lam, c_p, c_w,
                    E, _f32(np.repeat(base, C)))


@pytest.mark.parametrize("M,K,L", [(1, 9, 40), (2, 33, 40), (3, 129, 300), (64, 65, 1000),
                                   (2047, 5, 100), (2048, 5, 100), (2049, 5, 100), (5000, 3, 64)])
def test_flat_and_small_grids(ctx, dev, M, K, L):
    _check(ctx, dev, _workload(f"flat-{M}", L, K, lam_grid(M, 2.0 ** -10, 2.0 ** 7), 8))


@pytest.mark.parametrize("lo,hi", [(2.0 ** -10, 2.0 ** -9), (100.0, 128.0), (0.25, 0.2500008)])
def test_multipliers_on_one_side_of_the_costs(ctx, dev, lo, hi):
    lam = np.unique(lam_grid(20, lo, hi))
    _check(ctx, dev, _workload(f"side-{lo:g}", 500, 51, lam, 8))


def test_descending_multipliers_are_scanned(ctx, dev):
    _check(ctx, dev, _workload("descending", 300, 33, lam_grid(40)[::-1].copy(), 8))
