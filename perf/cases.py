"""Performance cases of the reservation path, through its public entry points.

Each case is one kind of call a program of this package makes:

  step      class_quantile, dro_cost_eval, dro_argmin_reservation: one pass of
            the whole dense path, as bench.py times it
  quantile  class_quantile alone (what an SAA or fixed-percentile reservation
            costs)
  table     dro_exact_table: the worst-case table and optimum from value
            counts, the call for programs that need only the results
  dual      dro_continuous_dual: the dual without a multiplier grid
  policy    policies.table: every policy's reservation, priced on shifted sets
  solve     serving.dro_bcd_solve: Alg. 1 around the reservation update
  block     bcd_block_step: one capacity-constrained reservation update

Samples are heavy-tailed output lengths drawn on the GPU from the seed alone,
with the distributions of workloads/configs.py; segment sizes follow from the
case, so that another seed means new data of the same shape (drifting traffic).
One Context serves a process, as in bench.py.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

import paper_2607_16892_amd as dro
from paper_2607_16892_amd import policies, serving
from workloads import eta_grid, fit_lognormal, lam_grid, TRACE_STATS
from workloads.configs import serving_workload

DEV = "cuda:0"
BINS = 32769            # sample values 0 .. 2^15
FRACS = (0.0, 0.05, 0.1, 0.15, 0.2, 0.3, 0.5)   # radii of the policy comparison, x mean
RHOS = (2, 5, 10, 20, 50, 100)
SHIFTS = (1.0, 1.5, 2.0, 2.5, 3.0)


def _case(kind, name=None, *, segs=1, ratios=1, n=1000, ragged=False, L=4096, K=64, M=32, E=1,
          dist="lognormal", G=0, J=0):
    c = dict(kind=kind, segs=segs, ratios=ratios, n=n, ragged=ragged, L=L, K=K, M=M, E=E,
             dist=dist, G=G, J=J)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one class of 1,000 lengths: a small service's reservation, bound by launches
        _case("step", "step-1x1k", n=1000, L=4096, K=64, M=32),
        # classes of very different traffic on grids of odd sizes, three radii
        _case("step", "step-6-ragged", segs=6, n=120_001, ragged=True, L=6000, K=333, M=50, E=3),
        # four classes of 100,000 lengths: one re-optimisation of a mid-size service
        _case("step", "step-4x100k", segs=4, n=100_000, L=8192, K=512, M=128),
        # the benchmark's 16 classes of a million lengths
        _case("step", "step-16x1M", segs=16, n=1_000_000, L=32768, K=2048, M=256, dist="mixture"),
        # critical-fractile reservations of the same data, and of many unequal classes
        _case("quantile", "quantile-16x1M", segs=16, n=1_000_000, L=32768, dist="mixture"),
        _case("quantile", "quantile-40-ragged", segs=40, n=200_003, ragged=True, L=8192),
        # the table by value counts: the benchmark's classes, and the regime sweep of
        # 16 cost ratios x 16 radii over shared segments
        _case("table", "table-16x1M", segs=16, n=1_000_000, L=32768, K=2048, M=256, dist="mixture"),
        _case("table", "table-8x250k-sweep", segs=8, ratios=16, n=250_000, L=32768, K=1024, M=128,
              E=16),
        # the grid-free dual of the benchmark's classes
        _case("dual", "dual-16x1M", segs=16, n=1_000_000, L=32768, K=2048, M=256, dist="mixture"),
        # 15 policies priced on five shifted sets, every integer reservation a candidate
        _case("policy", "policy-1M", segs=1, n=1_000_000, L=8192, K=8193, M=256),
        # Alg. 1 over 12 (TP, PP) configurations of 48 GPUs
        _case("solve", "solve-15x100k", segs=15, n=100_000, L=8192, K=2048, M=256, G=12, J=48),
        # one block step under six groups' KV capacities
        _case("block", "block-8x400k", segs=8, n=400_000, L=32768, K=1024, M=128, G=6),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step"] * 4 + ["quantile"] * 2 + ["table"] * 2 + ["dual", "policy", "solve",
                                                                        "block"])
    ragged = rng.random() < 0.5
    dist = rng.choice(["lognormal", "mixture"])
    L = log(500, 32768)
    if kind == "policy":
        L = log(500, 8192)
        return _case(kind, n=log(5_000, 1_000_000), L=L, K=L + 1, M=log(32, 256))
    if kind == "solve":
        return _case(kind, segs=rng.randint(3, 15), n=log(2_000, 100_000), L=8192,
                     K=log(128, 2048), M=log(32, 256), G=12, J=rng.randint(16, 48))
    segs, n = log(1, 32), log(500, 1_000_000)
    n = max(500, min(n, 16_000_000 // segs))
    if kind == "quantile":
        return _case(kind, segs=segs, n=n, ragged=ragged, L=L, dist=dist)
    K, M = min(log(16, 2048), L), log(8, 256)
    if kind == "table":
        ratios = rng.choice([1, 1, 2, 5, 16])
        E = rng.choice([1, 1, 3, 16])
        K = max(16, min(K, 16_777_216 // (segs * ratios * M)))
        return _case(kind, segs=segs, ratios=ratios, n=n, ragged=ragged, L=L, K=K, M=M, E=E,
                     dist=dist)
    K = max(16, min(K, 8_388_608 // (segs * M), int(2e12 / (segs * n * M))))
    if kind == "dual":
        return _case(kind, segs=segs, n=n, ragged=ragged, L=L, K=K, M=M, E=rng.choice([1, 1, 4]),
                     dist=dist)
    if kind == "block":
        K = max(16, min(K, int(5e11 / (segs * n * M))))
        return _case(kind, segs=segs, n=n, ragged=ragged, L=L, K=K, M=M, G=rng.randint(1, 8),
                     dist=dist)
    return _case(kind, segs=segs, n=n, ragged=ragged, L=L, K=K, M=M, E=rng.choice([1, 1, 1, 3]),
                 dist=dist)


# ------------------------------------------------------------------ inputs ----

def _sizes(case):
    """Samples of each segment: equal, or spread over a factor of 16."""
    n, S = case["n"], case["segs"]
    if not case["ragged"]:
        return [n] * S
    return [max(1, int(n * 16.0 ** -((0.6180339887 * s) % 1.0))) for s in range(S)]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1_000_003 * (int(seed) + 1))
    return g


def _samples(case, seed):
    """int32 lengths in [1, L], segment after segment, on the GPU."""
    g, L, S = _gen(seed), case["L"], case["segs"]
    rng = np.random.default_rng(int(seed))
    top = L / 8.0
    parts = []
    for s, n in enumerate(_sizes(case)):
        def logn(mean, sigma):
            z = torch.randn(n, generator=g, device=DEV)
            return torch.exp(z * sigma + (math.log(mean) - 0.5 * sigma * sigma))

        if case["dist"] == "mixture":   # 0.7/0.3 lognormal mixture, 2 % Lomax(1.5) tail
            m1, m2 = rng.uniform(L / 1600.0 + 1.0, L / 11.0 + 1.0, 2)
            x = torch.where(torch.rand(n, generator=g, device=DEV) < 0.7, logn(m1, 1.0),
                            logn(m2, 1.0))
            u = torch.rand(n, generator=g, device=DEV).clamp_min_(1e-7)
            tail = torch.rand(n, generator=g, device=DEV) < 0.02
            x = torch.where(tail, max(m1, m2) * u.pow(-1.0 / 1.5), x)
        else:                           # class means log-spaced up to L / 8
            lo = max(5.0, top / 100.0)
            mean = lo * (top / lo) ** (s / max(S - 1, 1)) * rng.uniform(0.9, 1.1)
            x = logn(mean, float(rng.uniform(0.8, 1.2)))
        parts.append(x.round_().clamp_(1, L).to(torch.int32))
    return torch.cat(parts)


@functools.lru_cache(maxsize=64)
def _arrays(kind, segs, ratios, sizes, L, K, M):
    """Offsets, segment map, grids and support bounds of a case (the same for every seed)."""
    off = np.zeros(segs + 1, np.int64)
    off[1:] = np.cumsum(sizes)
    C = segs * ratios
    seg = None if ratios == 1 else (np.arange(C) % segs).astype(np.int32)
    return off, seg, np.full(C, L, np.int32), eta_grid(K, L), lam_grid(M)


def _costs(case, seed):
    """(c_p, c_w): ratios in [1, 128] over shared segments, else log-uniform in [2, 64]."""
    S, R = case["segs"], case["ratios"]
    if R > 1:
        rho = 128.0 ** (np.arange(R) / (R - 1))
        return np.float32(0.5 * np.repeat(rho, S)), np.full(S * R, 0.5, np.float32)
    rng = np.random.default_rng(int(seed) + 77)
    return np.float32(np.exp(rng.uniform(math.log(2.0), math.log(64.0), S))), np.ones(S, np.float32)


def _radii(case, xi):
    """eps [E*C] fp32 on the GPU: 2 % of the class mean, or E radii from 0 to 20 %."""
    E, S, R = case["E"], case["segs"], case["ratios"]
    means = torch.stack([p.to(torch.int64).sum() / n for p, n in
                         zip(torch.split(xi, _sizes(case)), _sizes(case))]).double().repeat(R)
    f = [0.02] if E == 1 else [0.2 * e / (E - 1) for e in range(E)]
    return torch.cat([(means * x).float() for x in f])


def _groups(case, seed):
    rng = np.random.default_rng(int(seed) + 99)
    C, G = case["segs"], case["G"]
    mask = rng.random((C, G)) < 0.5
    mask[np.arange(C), rng.integers(G, size=C)] = True
    conc = np.where(mask, rng.uniform(0.5, 4.0, (C, G)), 0.0).astype(np.float32)
    cap = rng.uniform(0.6 * case["L"], 12.0 * case["L"], G).astype(np.float32)
    return cap, conc.reshape(-1), float(np.float32(0.2))


_CTX = []


def _ctx():
    if not _CTX:
        _CTX.append(dro.Context(0))
    return _CTX[0]


def _policy_inputs(case, seed):
    g = _gen(seed)
    mu, sigma = fit_lognormal(*TRACE_STATS["burst"])
    n, L = case["n"], case["L"]

    def draws():
        return torch.exp(torch.randn(n, generator=g, device=DEV) * sigma + mu)

    x = draws().round_().clamp_(1, L).to(torch.int32)
    y = draws()
    xe = torch.cat([(s * y).round_().clamp_(1, L).to(torch.int32) for s in SHIFTS])
    mean = float(x.to(torch.int64).sum()) / n
    return x, xe, mean


def _problem(offsets, xi, L, eta, lam, c_p, c_w, seg):
    p = dro.Problem.from_arrays(DEV, offsets, np.zeros(0, np.int32), L, eta, lam, c_p, c_w, seg=seg)
    p.xi = xi
    return p


def prepare(case, seed):
    kind = case["kind"]
    st = dict(kind=kind, ctx=_ctx())
    if kind == "solve":
        w, svc = serving_workload(C=case["segs"], N=case["n"], J=case["J"], L=case["L"],
                                  K=case["K"], M=case["M"], seed=int(seed) + 6)
        st.update(prob=dro.Problem.from_workload(w, DEV), svc=serving.Service.from_model(svc, DEV),
                  eps=torch.from_numpy(w.eps.copy()).to(DEV), z0=torch.from_numpy(svc.z0).to(DEV))
        return st
    if kind == "policy":
        x, xe, mean = _policy_inputs(case, seed)
        n, L, nr, ns = case["n"], case["L"], len(RHOS), len(SHIFTS)
        eta, lam = eta_grid(case["K"], L), lam_grid(case["M"])
        ones = np.ones(nr * ns, np.float32)
        st["train"] = _problem(np.array([0, n], np.int64), x, np.full(nr, L, np.int32), eta, lam,
                               np.float32(RHOS), ones[:nr], np.zeros(nr, np.int32))
        st["evalp"] = _problem(np.arange(ns + 1, dtype=np.int64) * n, xe,
                               np.full(nr * ns, L, np.int32), eta, lam, np.float32(RHOS * ns), ones,
                               np.repeat(np.arange(ns), nr).astype(np.int32))
        st["eps"] = torch.tensor([f * mean for f in FRACS for _ in RHOS], dtype=torch.float32,
                                 device=DEV)
        return st
    off, seg, L, eta, lam = _arrays(kind, case["segs"], case["ratios"], tuple(_sizes(case)),
                                    case["L"], case["K"], case["M"])
    xi = _samples(case, seed)
    st["prob"] = _problem(off, xi, L, eta, lam, *_costs(case, seed), seg)
    st["eps"] = _radii(case, xi)
    if kind == "block":
        st["groups"] = dro.Groups.from_numpy(*_groups(case, seed), DEV)
        st["k"] = dro.bcd_init_state(st["ctx"], st["prob"])
    return st


def run(st):
    kind, ctx = st["kind"], st["ctx"]
    if kind == "step":
        q = dro.class_quantile(ctx, st["prob"])
        r = dro.dro_cost_eval(ctx, st["prob"], st["eps"])
        a = dro.dro_argmin_reservation(ctx, st["prob"], st["eps"], r["S"])
        return dict(quantile=q, table=r, optimum=a)
    if kind == "quantile":
        return dro.class_quantile(ctx, st["prob"])
    if kind == "table":
        return dro.dro_exact_table(ctx, st["prob"], st["eps"])
    if kind == "dual":
        return dro.dro_continuous_dual(ctx, st["prob"], st["eps"])
    if kind == "policy":
        t = policies.table(ctx, st["train"], st["evalp"], st["eps"], FRACS)
        return {k: t[k] for k in ("eta", "cost", "cover", "cost_train", "cover_train")}
    if kind == "solve":
        return serving.dro_bcd_solve(ctx, st["prob"], st["eps"], st["svc"], st["z0"])
    return dro.bcd_block_step(ctx, st["prob"], st["eps"], st["groups"], st["k"])


# -------------------------------------------------------------------- work ----

def work(case):
    """Each input read once, each output written once; operations: two (a difference and
    its sum) per (class, reservation, multiplier, sample) term where the call evaluates
    every term by its definition, else the counts the results follow from."""
    kind, K, M, E = case["kind"], case["K"], case["M"], case["E"]
    sizes = _sizes(case)
    N, C = sum(sizes), case["segs"] * case["ratios"]
    terms = float(N) * case["ratios"] * K * M
    small = 4.0 * (K + M + 3 * C + E * C)
    if kind == "step":
        return dict(bytes=4.0 * N + small + 8.0 * C * K * M + 12.0 * E * C * K + 12.0 * C +
                    16.0 * E * C, flops=2 * terms)
    if kind == "block":
        return dict(bytes=4.0 * N + small + 17.0 * C, flops=2 * terms)
    if kind == "quantile":
        return dict(bytes=4.0 * N + 20.0 * C, flops=float(N))
    if kind == "table":
        return dict(bytes=4.0 * N + small + 12.0 * E * C * K + 16.0 * E * C,
                    flops=N + 10.0 * E * C * K * math.log2(M + 1))
    if kind == "dual":
        return dict(bytes=4.0 * N + small + 16.0 * E * C * K, flops=N + 20.0 * E * C * K * 16)
    if kind == "policy":
        nr, ns, R = len(RHOS), len(SHIFTS), len(FRACS) + 8
        return dict(bytes=4.0 * N * (1 + ns) + 4.0 * (K + M) + 16.0 * R * nr * (1 + ns),
                    flops=N * (1.0 + ns) + 10.0 * len(FRACS) * nr * K * math.log2(M + 1))
    gpus = [t * p for t in (1, 2, 4, 8) for p in (1, 2, 4)]
    ways = [1] * (case["J"] + 1)
    for gp in gpus:
        ways = [sum(ways[b - u * gp] for u in range(b // gp + 1)) for b in range(case["J"] + 1)]
    return dict(bytes=4.0 * N + small + 8.0 * C * K,
                flops=N + 10.0 * C * K * math.log2(M + 1) + 6.0 * ways[-1] * C * len(gpus))


def tolerance(case):
    # the library defines its sums, tables, optima and quantiles exactly
    if case["kind"] == "dual":
        # fp64: W to round-off (8e-17 seen); the minimising gamma solves x0(gamma) = an integer
        # x0 = L/2 + (B - C)/(2 gamma), whose rounding moves gamma by x0 / |x0 - L/2| <= 2^16
        # units in the last place at the worst grid point
        return {"rel": 1e-12, "max": 6e-11}
    if case["kind"] == "solve":     # fp64 simplex: vertices to round-off, decisions exactly
        return {"rel": 1e-12, "max": 1e-11}
    return "exact"


# ----------------------------------------------------- results in 64 bits ----

def _prefix(xi):
    """fp64 #{x <= v} and sum{x : x <= v} for v = 0 .. 2^15 (exact integers)."""
    h = torch.bincount(xi, minlength=BINS).double()
    v = torch.arange(BINS, device=DEV, dtype=torch.float64)
    return h.cumsum(0), (h * v).cumsum(0)


def _sums(pre, N, L, eta, g, cp, cw):
    """S for eta [K, 1] and multipliers g (broadcast): phi is the larger of two lines in x."""
    cn, sm = pre
    B, C = cw * eta, cp * (L - eta)
    a1, a2 = torch.clamp(g, max=cw), torch.clamp(g, max=cp)
    t = torch.floor((B - C + a2 * L) / (a1 + a2)).clamp(-1, L).long()
    n1 = torch.where(t >= 0, cn[t.clamp_min(0)], 0.0)
    s1 = torch.where(t >= 0, sm[t.clamp_min(0)], 0.0)
    return B * n1 - a1 * s1 + (C - a2 * L) * (N - n1) + a2 * (sm[-1] - s1)


def _table64(xi, L, eta, lam, cp, cw, eps, keep_S=False):
    """(S [K, M] or None, W [E, K]) of one class with radii eps [E]."""
    pre, N = _prefix(xi), xi.numel()
    S = _sums(pre, N, float(L), eta.double()[:, None], lam.double()[None, :], cp, cw)
    W = torch.stack([(S / N + lam.double() * e).amin(1) for e in eps.double()])
    return (S if keep_S else None), W


def _rank64(xi, cp, cw):
    N = xi.numel()
    j = min(N, max(1, math.ceil(cp * N / (cp + cw))))
    return int(torch.sort(xi)[0][j - 1]), j


def _dual64(xi, L, eta, cp, cw, eps):
    """(W, gamma) [E, K] by bisection of the right derivative over [0, max(c_p, c_w)]."""
    (cn, sm), N = _prefix(xi), xi.numel()
    eta = eta.double()[None, :]
    ev = eps.double()[:, None].expand(-1, eta.shape[1])
    B, C = cw * eta, cp * (L - eta)

    def at(g):
        a1, a2 = torch.clamp(g, max=cw), torch.clamp(g, max=cp)
        far = torch.where(B >= C, L + 2.0, -2.0).double()   # parallel lines at g = 0
        x0 = torch.where(a1 + a2 > 0, (B - C + a2 * L) / (a1 + a2), far).clamp(-2, L + 2)
        t = torch.floor(x0)
        i = t.long().clamp(0, L)
        n1, s1 = torch.where(t >= 0, cn[i], 0.0), torch.where(t >= 0, sm[i], 0.0)
        J = g * ev + (B * n1 - a1 * s1 + (C - a2 * L) * (N - n1) + a2 * (sm[-1] - s1)) / N
        tie = (t == x0) & (t >= 0) & (t <= L)
        p = (t.long() - 1).clamp(0, L)
        n0, s0 = torch.where(t >= 1, cn[p], 0.0), torch.where(t >= 1, sm[p], 0.0)
        nt = torch.where(tie, n1 - n0, 0.0)
        n1, s1 = torch.where(tie, n0, n1), torch.where(tie, s0, s1)
        w1, w2 = (g < cw).double(), (g < cp).double()
        n2, s2 = N - n1 - nt, sm[-1] - s1 - nt * t
        d = -w1 * s1 - w2 * (L * n2 - s2) + nt * torch.maximum(-w1 * t, -w2 * (L - t))
        return J, ev + d / N

    lo, hi = torch.zeros_like(ev), torch.full_like(ev, max(cp, cw))
    _, d0 = at(lo)
    for _ in range(70):
        mid = 0.5 * (lo + hi)
        _, d = at(mid)
        up = d >= 0
        hi, lo = torch.where(up, mid, hi), torch.where(up, lo, mid)
    g = torch.where(d0 >= 0, torch.zeros_like(hi), hi)
    return at(g)[0], g


def exact(case, seed):
    kind = case["kind"]
    if kind == "solve":     # the state after a loop of linear programs and a search: no closed value
        return None
    if kind == "policy":
        return _exact_policy(case, seed)
    off, seg, L, eta, lam = _arrays(kind, case["segs"], case["ratios"], tuple(_sizes(case)),
                                    case["L"], case["K"], case["M"])
    xi = _samples(case, seed)
    parts = torch.split(xi, _sizes(case))
    cps, cws = _costs(case, seed)
    C, L = case["segs"] * case["ratios"], case["L"]
    cp, cw = [float(v) for v in cps], [float(v) for v in cws]
    xs = [parts[c % case["segs"]] for c in range(C)]
    et, lm = torch.from_numpy(eta).to(DEV), torch.from_numpy(lam).to(DEV)
    if kind == "quantile":
        r = [_rank64(xs[c], cp[c], cw[c]) for c in range(C)]
        return dict(q_value=torch.tensor([q for q, _ in r], dtype=torch.int32),
                    q_rank=torch.tensor([j for _, j in r], dtype=torch.int64))
    eps = _radii(case, xi).view(case["E"], C)
    if kind == "dual":
        d = [_dual64(xs[c], L, et, cp[c], cw[c], eps[:, c]) for c in range(C)]
        return dict(W=torch.stack([w for w, _ in d], 1), gamma=torch.stack([g for _, g in d], 1))
    t = [_table64(xs[c], L, et, lm, cp[c], cw[c], eps[:, c], kind == "step") for c in range(C)]
    W = torch.stack([w for _, w in t], 1)
    if kind == "table":
        return dict(W=W, m_star=None, k_star=None, W_star=W.amin(2), m_at_star=None)
    if kind == "step":
        return dict(quantile=None, table=dict(S=torch.stack([s for s, _ in t]), W=W, m_star=None),
                    optimum=dict(k_star=None, W_star=W.amin(2), m_at_star=None))
    # the block step's sweep: each class's best admissible reservation given the others
    cap, conc, kappa = _groups(case, seed)
    conc = conc.reshape(C, case["G"]).astype(np.float64)
    eta64 = eta.astype(np.float64)
    Wh = W[0].cpu().numpy()
    means = [float(x.to(torch.int64).sum()) / x.numel() for x in xs]
    k = [max(0, int(np.searchsorted(eta, m, side="right")) - 1) for m in means]
    w_star = []
    for c in range(C):
        others = sum(conc[d] * eta64[k[d]] for d in range(C) if d != c)
        g = conc[c] > 0
        room = ((cap[g] - (1 + kappa) * (others[g] if C > 1 else 0.0)) /
                ((1 + kappa) * conc[c][g])).min()
        top = max(0, int(np.searchsorted(eta64, room, side="right")) - 1)
        k[c] = int(Wh[c, :top + 1].argmin())
        w_star.append(Wh[c, k[c]])
    use = (1 + kappa) * sum(conc[c] * eta64[k[c]] for c in range(C))
    return dict(k_next=None, W_star=torch.tensor(w_star, dtype=torch.float64), q_value=None,
                usage=torch.from_numpy(use), feasible=None)


def _exact_policy(case, seed):
    x, xe, mean = _policy_inputs(case, seed)
    L, n = case["L"], case["n"]
    eta = torch.arange(L + 1, device=DEV, dtype=torch.int32)   # K = L + 1: every integer
    lam = torch.from_numpy(lam_grid(case["M"])).to(DEV)
    eps = torch.tensor([f * mean for f in FRACS], dtype=torch.float32, device=DEV)
    best = torch.stack([_table64(x, L, eta, lam, float(r), 1.0, eps)[1].argmin(1) for r in RHOS], 1)
    srt = torch.sort(x)[0]

    def q(a, b):
        return srt[max(1, -(-a * n // b)) - 1].long()

    s1, s2 = int(x.long().sum()), int(x.long().square().sum())
    sd = math.sqrt(n * s2 - s1 * s1)
    fixed = [q(9, 10), -(-q(19, 20) // 16) * 16, q(99, 100), -(-s1 // n), L] + \
        [min(L, math.ceil((s1 + k * sd) / n)) for k in (1, 2)]
    rows = [best[e] for e in range(len(FRACS))] + [torch.stack([q(r, r + 1) for r in RHOS])] + \
        [torch.full((len(RHOS),), int(v), device=DEV) for v in fixed]
    res = torch.stack(rows).double()                            # [R, rhos]
    rho = torch.tensor(RHOS, dtype=torch.float64, device=DEV)

    def price(y):
        cn, sm = _prefix(y)
        i = res.long()
        return (rho * ((sm[-1] - sm[i]) - res * (n - cn[i])) + (res * cn[i] - sm[i])) / n

    return dict(eta=None, cost=torch.stack([price(y) for y in torch.split(xe, n)], 1), cover=None,
                cost_train=price(x), cover_train=None)
