"""Alg. 1 at the sizes where its kernels change how they work: the sweep with and
without its operands in LDS, the routing LP and the fused Blocks 1-2 with the
tableau in LDS and in memory, the configuration search with its tables in LDS and
in memory, its waits kept and looked up, with one and with several configurations
per thread.  Bars as in test_serving_gpu: everything but the LP in the same
fixed-order arithmetic, bit for bit; the LP's objective to 1e-9 relative and its
routing to 1e-7."""
import numpy as np
import pytest

import oracle
from oracle import serving as osv
from workloads import random_workload
from workloads.configs import serving_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


def _t(a, dt, dev):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=dt)).to(dev)


def _bits(a):
    return np.ascontiguousarray(a, np.float64).view(np.uint64)


# (C, K, G): one grid point; a last piece of the 64-way search; operands one step
# inside LDS (C G + C + G = 3,071) and beyond it; a grid beyond LDS (K > 6,144);
# more configurations than lanes
@pytest.mark.parametrize("C,K,G", [(1, 1, 1), (3, 65, 2), (31, 64, 95), (32, 129, 95), (2, 6145, 2),
                                   (3, 257, 130)])
@pytest.mark.parametrize("tight", [1.0, 0.3, 0.0])
def test_block_step_sweep_paths(ctx, dev, C, K, G, tight):
    import torch
    import paper_2607_16892_amd as dro
    w = random_workload(seed=C + K + G, C=C, N=40, L=max(600, K + 55), K=K, M=5, E=1,
                        with_groups=True, G=G)
    cap = w.groups.cap * np.float32(tight)  # 0: no reservation is feasible
    w.groups.cap[:] = cap
    print(f"[gpu] sweep C={C} K={K} G={G} tight={tight}", flush=True)
    k_prev = np.random.default_rng(K).integers(0, K, C).astype(np.int32)
    grp = dro.Groups.from_numpy(w.groups.cap, w.groups.conc, w.groups.kappa, dev)
    g = dro.bcd_block_step(ctx, dro.Problem.from_workload(w, dev), _t(w.eps[:C], np.float32, dev),
                           grp, _t(k_prev, np.int32, dev))
    torch.cuda.synchronize()
    W, _ = oracle.W_table(w, oracle.S_exact(w))
    o = oracle.bcd_step(w, W[0], k_prev)
    g = {k: v.cpu().numpy() for k, v in g.items()}
    assert np.array_equal(g["k_next"], o["k_next"])
    assert np.array_equal(g["feasible"], o["feasible"])
    assert np.array_equal(_bits(g["W_star"]), _bits(o["W_star"]))
    assert np.array_equal(_bits(g["usage"]), _bits(o["usage"]))


# tableaus of 6,230 and 26,195 doubles (LDS holds 19,456)
@pytest.mark.parametrize("C,seed", [(11, 21), (26, 22)])
def test_alg1_tableau_in_lds_and_in_memory(ctx, dev, C, seed):
    import torch
    import paper_2607_16892_amd as dro
    from paper_2607_16892_amd import serving as gs
    w, svc = serving_workload(C=C, N=2000, J=20, K=129, M=16, seed=seed)
    print(f"[gpu] solve C={C} G={svc.G}", flush=True)
    s = gs.Service.from_model(svc, dev)
    T, ET2 = osv.service_times(svc, w)
    z = np.ones(svc.G, np.int32)
    z[3] = 0
    zero = np.zeros((C, svc.G))
    eta_c = np.full(C, 150, np.int32)
    mem = osv.memory(svc, T, zero, z, eta_c, zero.astype(np.uint8))
    Wq = osv.queue(svc, T, ET2, zero, z, mem)
    Wc = np.random.default_rng(seed).uniform(50.0, 3000.0, C)
    ref_pi, ref_obj = osv.routing_lp(svc, Wc, T, Wq, z, eta_c, zero.astype(np.uint8))
    r = gs.bcd_routing_lp(ctx, C, s, _t(Wc, np.float64, dev), _t(T, np.float64, dev),
                          _t(Wq, np.float64, dev), _t(z, np.int32, dev), _t(eta_c, np.int32, dev),
                          _t(zero, np.uint8, dev))
    torch.cuda.synchronize()
    assert r["info"].cpu().numpy()[1] == 0
    assert abs(float(r["objective"].cpu()[0]) - ref_obj) <= 1e-9 * abs(ref_obj)
    assert np.max(np.abs(r["pi"].cpu().numpy() - ref_pi)) <= 1e-7
    # the whole loop at that size, its launch sizing included
    ref = osv.solve(w, svc)
    g = gs.dro_bcd_solve(ctx, dro.Problem.from_workload(w, dev), _t(w.eps[:C], np.float32, dev), s,
                         svc.z0)
    torch.cuda.synchronize()
    assert np.array_equal(g["z"].cpu().numpy(), ref["z"])
    assert np.array_equal(g["k"].cpu().numpy(), ref["k"])
    assert np.array_equal(g["delta"].cpu().numpy(), ref["delta"])
    assert np.max(np.abs(g["pi"].cpu().numpy() - ref["pi"])) <= 1e-7
    assert (g["info"]["outer"], g["info"]["inner"]) == (ref["outer"], ref["inner"])


# two z, a part of a block, many blocks (the tables in LDS, one z per thread), 811,801 z
# (four per thread, the tables beyond LDS); 32 configurations, whose waits are looked up:
# tables in LDS, and beyond it; classes in more than one tile of the sums (1,024 entries)
@pytest.mark.parametrize("C,J,configs", [(5, 1, [(1, 1)]), (5, 37, [(1, 1), (2, 1), (4, 2)]),
                                         (5, 170, [(1, 1), (2, 1), (4, 1)]),
                                         (5, 1800, [(1, 1), (2, 1)]),
                                         (5, 40, [(4, 2), (8, 2), (4, 4), (8, 4)] * 8),
                                         (33, 40, [(4, 2), (8, 2), (4, 4), (8, 4)] * 8),
                                         (171, 10, None), (86, 10, None), (85, 10, None)])
@pytest.mark.parametrize("routed", ["all", "none of the last", "nothing"])
def test_config_search_paths(ctx, dev, C, J, configs, routed):
    import torch
    from paper_2607_16892_amd import serving as gs
    w, svc = serving_workload(C=C, N=500, J=J, K=65, M=8, configs=configs, seed=J)
    s = gs.Service.from_model(svc, dev)
    print(f"[gpu] config search J={J} G={svc.G} routed={routed}", flush=True)
    T, ET2 = osv.service_times(svc, w)
    rng = np.random.default_rng(J)
    pi = rng.dirichlet(np.ones(svc.G + 1), C)[:, :svc.G] * 0.3
    pi[2] = 0.0                       # a class that is not served
    if routed != "all":
        pi[:, -1] = 0.0               # counts that change nothing: ties go to the first z
    if routed == "nothing":
        pi[:] = 0.0
    delta = (rng.random((C, svc.G)) < 0.2).astype(np.uint8)
    eta_c = rng.integers(0, 60, C).astype(np.int32)
    Wc = rng.uniform(50.0, 3000.0, C)
    zb, best, rank, nfeas = osv.config_search_vec(svc, Wc, T, ET2, pi, eta_c, delta)
    zt = _t(svc.z0, np.int32, dev)
    r = gs.bcd_config_search(ctx, C, s, _t(Wc, np.float64, dev), _t(T, np.float64, dev),
                             _t(ET2, np.float64, dev), _t(pi, np.float64, dev),
                             _t(eta_c, np.int32, dev), _t(delta, np.uint8, dev), zt)
    torch.cuda.synchronize()
    assert int(r["n_feasible"].cpu()[0]) == nfeas
    if nfeas:
        assert int(r["best_rank"].cpu()[0]) == rank
        assert _bits(r["best_objective"].cpu().numpy())[0] == _bits(np.array([best]))[0]
    keep = nfeas == 0 or osv.feasible(svc, T, pi, svc.z0, eta_c, delta) and \
        osv.state_objective(svc, Wc, T, ET2, pi, svc.z0, eta_c, delta) == best
    assert np.array_equal(zt.cpu().numpy(), svc.z0 if keep else zb)
