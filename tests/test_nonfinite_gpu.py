"""Hot calls do not check device data, so a radius, an S or a W that is infinite or
NaN reaches the minima.  Where no value is below infinity the result is infinity
at the last index searched (inside the table), and the rows beside it are what
they are without it, bit for bit.  A support bound outside [0, 2^15] leaves the
other classes' rows as they are too (lookups stay inside the value counts).
"""
import numpy as np
import pytest

from workloads.configs import random_workload

pytestmark = pytest.mark.gpu

INF, NAN = float("inf"), float("nan")


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


def _check(rows, ref, bad, M, kmax):
    """rows: outputs with the radius rows `bad` not finite; ref: without those rows."""
    import torch
    good = [e for e in range(rows["W_star"].shape[0]) if e not in bad]
    for k in ("W", "m_star", "k_star", "W_star", "m_at_star"):
        assert torch.equal(rows[k][good], ref[k]), k
    for e in bad:
        assert bool((rows["W"][e] == INF).all()) and bool((rows["W_star"][e] == INF).all())
        assert bool((rows["m_star"][e] == M - 1).all()) and bool((rows["m_at_star"][e] == M - 1).all())
        assert torch.equal(rows["k_star"][e], kmax)


# (K past a block of the argmin, M past the staged multipliers, radii past a wave)
@pytest.mark.parametrize("K,M,E", [(9, 4, 4), (1, 1, 5), (1500, 3, 4), (5, 2050, 6), (40, 30, 80)])
def test_radii_that_are_not_finite(ctx, dev, K, M, E):
    import torch
    import paper_2607_16892_amd as dro
    w = random_workload(seed=K + M, C=4, N=(60, 9, 300, 1), L=2000, K=K, M=M, E=E)
    prob = dro.Problem.from_workload(w, dev)
    eps = torch.from_numpy(w.eps.copy()).to(dev).view(E, w.C)
    bad = [1, E - 1]
    good = [e for e in range(E) if e not in bad]
    eps[1] = INF
    eps[E - 1] = NAN
    k_max = torch.tensor([K - 1, 0, K // 2, K + 7], dtype=torch.int32, device=dev)
    print(f"[gpu] non-finite radii: K={K} M={M} E={E}", flush=True)

    def run(e):
        e = e.contiguous().view(-1)
        d = dro.dro_cost_eval(ctx, prob, e)
        a = dro.dro_argmin_reservation(ctx, prob, e, d["S"], k_max=k_max)
        t = dro.dro_exact_table(ctx, prob, e, k_max=k_max)
        return dict(a, W=d["W"], m_star=d["m_star"]), t

    (rows, table), (ref, ref_table) = run(eps), run(eps[good])
    torch.cuda.synchronize()
    kmax = k_max.clamp(0, K - 1)
    _check(rows, ref, bad, M, kmax)
    _check(table, ref_table, bad, M, kmax)


def test_an_S_that_is_not_finite(ctx, dev):
    import torch
    import paper_2607_16892_amd as dro
    w = random_workload(seed=8, C=3, N=(60, 9, 300), L=500, K=33, M=11, E=2)
    prob = dro.Problem.from_workload(w, dev)
    eps = torch.from_numpy(w.eps.copy()).to(dev)
    S = dro.dro_cost_eval(ctx, prob, eps)["S"]
    ref = dro.dro_argmin_reservation(ctx, prob, eps, S)
    bad = S.clone()
    bad[0] = INF
    bad[1] = NAN
    got = dro.dro_argmin_reservation(ctx, prob, eps, bad)
    torch.cuda.synchronize()
    for k in ("k_star", "W_star", "m_at_star"):
        assert torch.equal(got[k][:, 2], ref[k][:, 2]), k
    assert bool((got["W_star"][:, :2] == INF).all())
    assert bool((got["k_star"][:, :2] == w.K - 1).all())
    assert bool((got["m_at_star"][:, :2] == w.M - 1).all())


def test_sweeps_over_a_row_that_is_not_finite(ctx, dev):
    import torch
    import paper_2607_16892_amd as dro
    from paper_2607_16892_amd import serving
    w = random_workload(seed=9, C=3, N=(60, 9, 300), L=500, K=33, M=11, E=1)
    prob = dro.Problem.from_workload(w, dev)
    eps = torch.from_numpy(w.eps.copy()).to(dev)
    eps[1] = INF
    # one group; class 1 may take up to 10.5 grid steps whatever the others take
    step = float(w.eta[1])
    conc = np.array([[0.0], [1.0], [0.0]], np.float32)
    cap = np.array([10.5 * step], np.float32)
    grp = dro.Groups.from_numpy(cap, conc.reshape(-1), 0.0, dev)
    st = dro.bcd_block_step(ctx, prob, eps, grp, dro.bcd_init_state(ctx, prob))
    W = dro.dro_exact_table(ctx, prob, eps)["W"][0].contiguous()
    k_in = torch.zeros(3, dtype=torch.int32, device=dev)
    sw = serving.bcd_reservation_sweep(ctx, W, prob.eta, torch.from_numpy(conc).double().to(dev),
                                       torch.from_numpy(cap).double().to(dev), 0.0, k_in)
    torch.cuda.synchronize()
    last = int(np.flatnonzero(w.eta <= 10.5 * step).max())
    Wh = W.cpu().numpy()
    for got in (st["k_next"], sw["k"]):
        assert int(got[1]) == last
        for c in (0, 2):
            assert int(got[c]) == int(Wh[c].argmin())
    assert float(st["W_star"][1]) == INF


def test_support_bounds_outside_the_limits(ctx, dev):
    import torch
    import paper_2607_16892_amd as dro
    w = random_workload(seed=10, C=4, N=(60, 9, 300, 77), L=500, K=33, M=11, E=2)
    prob = dro.Problem.from_workload(w, dev)
    eps = torch.from_numpy(w.eps.copy()).to(dev)

    def run():
        return dict(dual=dro.dro_continuous_dual(ctx, prob, eps)["W"],
                    table=dro.dro_exact_table(ctx, prob, eps)["W"],
                    dense=dro.dro_cost_eval(ctx, prob, eps)["W"])

    ref = run()
    prob.L = torch.tensor([500, -5, 500, 70_000], dtype=torch.int32, device=dev)
    got = run()
    torch.cuda.synchronize()
    for k in ref:
        assert torch.equal(got[k][:, [0, 2]], ref[k][:, [0, 2]]), k
