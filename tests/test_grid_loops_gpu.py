"""Launches whose size grows with the problem loop over their items or rows
with at most 2^20 blocks (so a grid stays below 2^32 work-items).  These tests
take each loop past one pass, against the oracle's exact definitions:

- dro_cost_eval and dro_argmin_reservation on C K = 67,143,681 rows of one
  multiplier (the pass over the rows, in both its forms: 64 rows per block,
  two passes; App. A Steps 3-5);
- dro_argmin_reservation on E C = 2^20 + 6 radius rows (the argmin, one
  block per row, two passes), from an exact S table drawn with many ties
  (Prop. 4.2; ties to the lowest k, then m);
- class_quantile on 2^20 + 5 classes (the select, one block per class), and
  class_moments and bcd_init_state on 2^22 + 9 (four per block);
- dro_cost_eval on a C K M = 276,891,648-entry table whose last class is
  long enough to be split, so that its sums are added to zeros past the
  2^28 items of one pass of the zero fill, checked at sampled entries that
  include the last ones (App. A Steps 4-5);
- 2^31 - 1 radius rows, the limit, of which the last step of a 32-bit loop
  index would pass its range.
"""
import numpy as np
import pytest

import oracle
from plan_cpu import workload_plan
from workloads.configs import Workload, _csr, _f32, eta_grid, lam_grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


def _costs(rng, C):
    choice = [(8.0, 1.0), (1.0, 1.0), (2.0 ** 7, 2.0 ** -10), (2.0 ** -10, 2.0 ** 7), (0.5, 3.0)]
    pick = rng.integers(len(choice), size=C)
    return _f32([choice[i][0] for i in pick]), _f32([choice[i][1] for i in pick])


def test_table_rows_past_one_pass(ctx, dev):
    import torch
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(30)
    C, K, M, L = 2049, 32769, 1, 32768
    assert C * K > 64 << 20
    parts = [rng.integers(0, L + 1, n).astype(np.int32) for n in (3, 5)]
    offsets, xi = _csr(parts)
    seg = (np.arange(C) % 2).astype(np.int32)
    c_p, c_w = _costs(rng, C)
    eps = _f32(rng.uniform(0.0, 50.0, C))
    w = Workload("rows", C, offsets, seg, xi, np.full(C, L, np.int32), eta_grid(K, L),
                 lam_grid(2, 0.5, 8.0)[:1], c_p, c_w, 1, eps)
    print(f"[gpu] table rows: C={C} K={K}", flush=True)
    prob = dro.Problem.from_workload(w, dev)
    e = torch.from_numpy(eps).to(dev)
    r = dro.dro_cost_eval(ctx, prob, e)
    a = dro.dro_argmin_reservation(ctx, prob, e, r["S"])
    torch.cuda.synchronize()
    S = r["S"].view(C, K)
    # entries of the last classes (past the first pass) and of all
    cs = np.concatenate([np.full(3000, C - 1), rng.integers(0, C, 3000)])
    ks = rng.integers(0, K, cs.size)
    ref = oracle.S_exact_at(w, cs, ks, np.zeros_like(cs)).to_double()
    got = S[torch.from_numpy(cs).to(dev), torch.from_numpy(ks).to(dev)].cpu().numpy()
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
    # with one multiplier W = RN(RN(lam eps) + RN(S / N)) at every row
    N = torch.tensor([3.0, 5.0], dtype=torch.float64, device=dev)[torch.from_numpy(seg).to(dev).long()]
    W = (float(w.lam[0]) * e.double())[:, None] + S / N[:, None]
    assert torch.equal(r["W"][0], W) and int(r["m_star"].abs().max()) == 0
    Wh = W.cpu().numpy()
    k = Wh.argmin(1)
    assert np.array_equal(a["k_star"][0].cpu().numpy(), k)
    assert np.array_equal(a["W_star"][0].cpu().numpy(), Wh[np.arange(C), k])
    assert int(a["m_at_star"].abs().max()) == 0


def test_argmin_rows_past_one_pass(ctx, dev):
    import torch
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(31)
    C, K, M, E, L = (1 << 19) + 3, 9, 2, 2, 1000
    offsets, xi = _csr([rng.integers(0, L + 1, 3).astype(np.int32),
                        rng.integers(0, L + 1, 5).astype(np.int32)])
    seg = (np.arange(C) % 2).astype(np.int32)
    c_p, c_w = _costs(rng, C)
    eps = _f32(rng.uniform(0.0, 50.0, E * C))
    eps[:C] = 0.0
    w = Workload("rows", C, offsets, seg, xi, np.full(C, L, np.int32), eta_grid(K, L),
                 lam_grid(M, 0.5, 8.0), c_p, c_w, E, eps)
    assert E * C > 1 << 20
    # an exact S table (units of 2^-33) with ties: values from a small set
    lo = (rng.integers(0, 64, (C, K, M)).astype(np.uint64) << np.uint64(36))
    S = oracle.ExactS(np.zeros((C, K, M), np.int64), lo)
    Sd = S.to_double()
    print(f"[gpu] argmin rows: C={C} K={K} M={M} E={E}", flush=True)
    prob = dro.Problem.from_workload(w, dev)
    a = dro.dro_argmin_reservation(ctx, prob, torch.from_numpy(eps).to(dev),
                                   torch.from_numpy(Sd).to(dev))
    torch.cuda.synchronize()
    Wr, msr = oracle.W_table(w, S)
    ks, ws = oracle.argmin(Wr)
    assert np.array_equal(a["k_star"].cpu().numpy(), ks)
    assert np.array_equal(a["W_star"].cpu().numpy().view(np.uint64), ws.view(np.uint64))
    e_i, c_i = np.meshgrid(np.arange(E), np.arange(C), indexing="ij")
    assert np.array_equal(a["m_at_star"].cpu().numpy(), msr[e_i, c_i, ks])


def test_quantile_classes_past_one_pass(ctx, dev):
    rng = np.random.default_rng(32)
    C, L = (1 << 20) + 5, 32768
    parts = [rng.integers(1, L + 1, n).astype(np.int32) for n in (50, 1, 77)]
    offsets, xi = _csr(parts)
    seg = (np.arange(C) % 3).astype(np.int32)
    c_p, c_w = _costs(rng, C)
    w = Workload("classes", C, offsets, seg, xi, np.full(C, L, np.int32), eta_grid(3, L),
                 lam_grid(2), c_p, c_w, 1, np.zeros(C, np.float32))
    import torch
    import paper_2607_16892_amd as dro
    print(f"[gpu] quantile classes: C={C}", flush=True)
    q = dro.class_quantile(ctx, dro.Problem.from_workload(w, dev))
    torch.cuda.synchronize()
    qv, qr = oracle.quantile(w)
    assert np.array_equal(q["q_rank"].cpu().numpy(), qr)
    assert np.array_equal(q["q_value"].cpu().numpy(), qv)


def test_moments_of_classes_past_one_pass(ctx, dev):
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(35)
    C, L = (1 << 22) + 9, 300
    parts = [rng.integers(1, L + 1, n).astype(np.int32) for n in (50, 1, 77)]
    offsets, xi = _csr(parts)
    seg = (np.arange(C) % 3).astype(np.int32)
    one = np.ones(C, np.float32)
    print(f"[gpu] moments: C={C}", flush=True)
    prob = dro.Problem.from_arrays(dev, offsets, xi, np.full(C, L, np.int32), eta_grid(5, L),
                                   lam_grid(2), one, one, seg=seg)
    m = dro.class_moments(ctx, prob)
    k0 = dro.bcd_init_state(ctx, prob).cpu().numpy()
    eta = eta_grid(5, L).astype(np.int64)
    for s, x in enumerate(parts):
        x = x.astype(np.int64)
        at = seg == s
        for k, v in (("count", len(x)), ("sum", x.sum()), ("sumsq", (x * x).sum()), ("xmax", x.max())):
            assert (m[k].cpu().numpy()[at] == v).all(), k
        assert (k0[at] == np.flatnonzero(eta * len(x) <= x.sum()).max()).all()


def test_cost_eval_table_past_one_pass(ctx, dev):
    import torch
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(33)
    C, K, M, E, L = 33, 4097, 2048, 1, 4096
    offsets, xi = _csr([rng.integers(0, L + 1, 3).astype(np.int32),
                        np.array([0, L, 17], np.int32),
                        rng.integers(0, L + 1, 70_000).astype(np.int32)])
    seg = (np.arange(C) % 2).astype(np.int32)
    seg[C - 1] = 2
    c_p, c_w = _costs(rng, C)
    eps = _f32(rng.uniform(0.0, 30.0, E * C))
    w = Workload("table", C, offsets, seg, xi, np.full(C, L, np.int32), eta_grid(K, L),
                 lam_grid(M, 2.0 ** -10, 2.0 ** 7), c_p, c_w, E, eps)
    n = C * K * M
    assert (C - 1) * K * M >= (1 << 20) * 256 and not workload_plan(w)["stored"]
    print(f"[gpu] cost eval table: C={C} K={K} M={M} ({n} entries)", flush=True)
    prob = dro.Problem.from_workload(w, dev)
    S = torch.full((C, K, M), float("nan"), dtype=torch.float64, device=dev)
    r = dro.dro_cost_eval(ctx, prob, torch.from_numpy(eps).to(dev), S=S)
    torch.cuda.synchronize()
    Sg = S.view(-1)
    # sampled entries, the last 4096 of the table among them
    idx = np.unique(np.concatenate([rng.integers(0, n, 3000), np.arange(n - 4096, n)]))
    cs, ks, ms = idx // (K * M), (idx // M) % K, idx % M
    ref = oracle.S_exact_at(w, cs, ks, ms).to_double()
    got = Sg[torch.from_numpy(idx).to(dev)].cpu().numpy()
    assert np.array_equal(got.view(np.uint64), ref.view(np.uint64))
    # whole W rows for a few (c, k), one of them the last
    Wg = r["W"].cpu().numpy()
    mg = r["m_star"].cpu().numpy()
    for c, k in ((0, 0), (7, 2048), (C - 1, K - 1)):
        S_row = oracle.S_exact_at(w, np.full(M, c), np.full(M, k), np.arange(M))
        N = int(offsets[seg[c] + 1] - offsets[seg[c]])
        J = [oracle.J(S_row.hi[m], S_row.lo[m], float(w.lam[m]), float(eps[c]), N) for m in range(M)]
        m_best = int(np.argmin(J))  # first index of the minimum
        assert Wg[0, c, k] == J[m_best] and mg[0, c, k] == m_best


def test_radius_rows_up_to_the_limit(dev):
    """E C = 2^31 - 1, the most the entry points take: every radius of a table of one
    class, one grid point and two multipliers (75 GB of tables in all), against the
    definition in torch's fp64, a part of the radii at a time."""
    import torch
    import paper_2607_16892_amd as dro
    from workloads.configs import random_workload
    E, step = (1 << 31) - 1, 1 << 28
    w = random_workload(seed=34, C=1, N=5, L=300, K=1, M=2, E=1)
    print(f"[gpu] {E} radius rows", flush=True)
    lam = w.lam.astype(np.float64)
    eps = torch.empty(E, dtype=torch.float32, device=dev)
    for a in range(0, E, step):
        eps[a:a + step] = (torch.arange(a, min(a + step, E), device=dev) % 999_983).float() / 1024.0

    def check(W, m):
        W, m = W.view(-1), m.view(-1)
        for a in range(0, E, step):
            e = eps[a:a + step].double()
            J0, J1 = e * lam[0] + q[0], e * lam[1] + q[1]
            assert torch.equal(W[a:a + step], torch.minimum(J0, J1)), a
            assert torch.equal(m[a:a + step] == 1, J1 < J0), a

    with dro.Context(dev.index or 0) as c:
        prob = dro.Problem.from_workload(w, dev)
        S = dro.dro_cost_eval(c, prob, eps[:1].contiguous())["S"]
        q = [float(v) / 5.0 for v in S.view(-1).cpu()]
        r = dro.dro_cost_eval(c, prob, eps, want_S=False)
        check(r["W"], r["m_star"])
        del r
        r = dro.dro_exact_table(c, prob, eps, want_argmin=False)
        check(r["W"], r["m_star"])
        del r
        r = dro.dro_argmin_reservation(c, prob, eps, S)
        check(r["W_star"], r["m_at_star"])
        assert int(r["k_star"].abs().max()) == 0
        del r
    del eps
    torch.cuda.empty_cache()
