"""The grid-free dual with four lanes a row (up to 32,768 rows) and with one: the
rows of one call, repeated in a call of more radii that takes the other path, have
the same bits, at costs on either side and equal, radii of zero, small, typical and
past every sample, constant and single samples; and a sample of rows agrees with
the piecewise-linear dual evaluated at every breakpoint in 64 bits."""
import numpy as np
import pytest

from workloads.configs import Workload, _csr, _f32, eta_grid, lam_grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


def _solve(ctx, dev, parts, L, K, c_p, c_w, radii):
    import torch
    import paper_2607_16892_amd as dro
    C, E = len(parts), len(radii)
    off, xi = _csr([p.astype(np.int32) for p in parts])
    eps = _f32(np.repeat(np.asarray(radii, np.float64), C))
    w = Workload(f"dual-{E}x{K}", C, off, None, xi, np.full(C, L, np.int32), eta_grid(K, L),
                 lam_grid(8), _f32(c_p), _f32(c_w), E, eps)
    print(f"[gpu] dual C={C} K={K} E={E} rows={E * C * K}", flush=True)
    r = dro.dro_continuous_dual(ctx, dro.Problem.from_workload(w, dev),
                                torch.from_numpy(w.eps).to(dev))
    torch.cuda.synchronize()
    return w, r["W"].cpu().numpy(), r["gamma"].cpu().numpy()


def _dual(x, eta, L, cp, cw, eps):
    """min over gamma >= 0 of gamma eps + mean sup: at a breakpoint or a cost."""
    B, Cc = cw * eta, cp * (L - eta)
    g = [0.0, cw, cp]
    for v in np.unique(x):
        # where B - a1 v = C - a2 (L - v), on each side of the smaller cost
        d = 2.0 * v - L
        if d:
            g.append((B - Cc) / d)
        if cw < cp and v < L:
            g.append((cw * v - B + Cc) / (L - v))
        if cp < cw and v > 0:
            g.append((B - Cc + cp * (L - v)) / v)
    g = np.array([q for q in g if 0.0 <= q <= max(cw, cp)])
    a1, a2 = np.minimum(g, cw)[:, None], np.minimum(g, cp)[:, None]
    return (g * eps + np.maximum(B - a1 * x, Cc - a2 * (L - x)).mean(1)).min()


@pytest.mark.parametrize("K,E", [(1, 6), (65, 6), (1365, 6), (1366, 6), (2048, 4)])
def test_four_lanes_and_one_agree(ctx, dev, K, E):
    rng = np.random.default_rng(K)
    L = 3000
    parts = [rng.integers(0, L + 1, 301), np.full(9, 700), np.array([L]),
             np.minimum(rng.lognormal(5.0, 1.0, 1000), L).round()]
    c_p, c_w = [8.0, 1.0, 3.0, 0.5], [1.0, 1.0, 2.0 ** -10, 4.0]
    radii = [0.0, 0.02 * L, 1e-6, 0.3 * L, 2.0 * L, 0.001 * L][:E]
    w, W, g = _solve(ctx, dev, parts, L, K, c_p, c_w, radii)
    reps = -(-32769 // (len(parts) * K * E)) + 1
    _, W2, g2 = _solve(ctx, dev, parts, L, K, c_p, c_w, radii * reps)
    n = W.size
    for q in range(reps):
        part = slice(q * n, (q + 1) * n)
        assert np.array_equal(W2.ravel()[part].view(np.uint64), W.ravel().view(np.uint64))
        assert np.array_equal(g2.ravel()[part].view(np.uint64), g.ravel().view(np.uint64))
    Wr = W.reshape(E, len(parts), K)
    for e in range(E):
        for c, x in enumerate(parts):
            for k in {0, K // 3, K - 1}:
                ref = _dual(x.astype(np.float64), float(w.eta[k]), float(L), c_p[c], c_w[c],
                            float(np.float32(radii[e])))
                # a dozen roundings of terms up to c L (fp64), J flat to first order in gamma
                assert abs(Wr[e, c, k] - ref) <= 1e-12 * (abs(ref) + L * max(c_p[c], c_w[c]))
