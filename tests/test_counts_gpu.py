"""The prefix counts and sums of the sample values, at the edges of the passes
that build them: one row of counts per segment and more rows than the pass has
waves (16), values on both sides of its runs (512 values), of the packed halves
(2^14) and 2^15 itself, segments with unequal row counts, and the merged
histogram that takes over beyond 200 rows of a segment, beyond 768 rows of
segments of 8 or more, and where the scratch cannot hold the rows.

dro_reservation_cost at every integer reservation reads every entry: cover is
the count and the cost follows from the sum, so both are compared exactly with
numpy's integers (costs of 1 and 1, where (cost N) is an integer below 2^53 and
the quotient's rounding is numpy's).  class_moments and bcd_init_state share
the rows: compared with numpy's integer sums.
"""
import numpy as np
import pytest

from workloads.configs import Workload, _csr, _f32, eta_grid, lam_grid, random_workload

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 127, 128, 511, 512, 1023, 16383, 16384, 16895, 16896, 32255, 32256, 32767, 32768]


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


# (the last three through the merged histogram: 202 rows of one segment, 214 of one beside
# two short ones, 806 of 13)
@pytest.mark.parametrize("sizes", [(1,), (15,), (16_385,), (20, 300_001, 1, 40_000),
                                   (600_000,) * 3, (1_100_000,), (12_900_000,),
                                   (3, 5_000_000, 40), (13_200_000,), (3, 14_000_000, 40),
                                   (4_000_000,) * 13])
def test_every_prefix_entry(ctx, dev, sizes):
    import torch
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(len(sizes) + sizes[0])
    parts = []
    for n in sizes:
        x = np.clip(np.rint(rng.lognormal(7.0, 2.0, n)), 0, 32768).astype(np.int32)
        x[: len(EDGES)] = EDGES[:n]
        parts.append(rng.permutation(x))
    C = len(parts)
    off, xi = _csr(parts)
    w = Workload("counts", C, off, None, xi, np.full(C, 32768, np.int32), eta_grid(2049, 32768),
                 lam_grid(2), _f32([1] * C), _f32([1] * C), 1, np.zeros(C, np.float32))
    prob = dro.Problem.from_workload(w, dev)
    v = np.arange(-1, 32770, dtype=np.int32)
    print(f"[gpu] prefix entries of segments of {sizes}", flush=True)
    r = dro.dro_reservation_cost(ctx, prob, torch.from_numpy(np.repeat(v, C)).to(dev))
    m = dro.class_moments(ctx, prob)
    k0 = dro.bcd_init_state(ctx, prob)
    torch.cuda.synchronize()
    cover, cost = r["cover"].cpu().numpy(), r["cost"].cpu().numpy()
    for c, x in enumerate(parts):
        x64, n = x.astype(np.int64), len(x)
        h = np.bincount(x, minlength=32769).astype(np.int64)
        cnt = np.concatenate([[0], np.cumsum(h), [n]])
        sm = np.concatenate([[0], np.cumsum(h * np.arange(32769)), [x64.sum()]])
        assert np.array_equal(cover[:, c], cnt)
        S = (x64.sum() - sm) - v * (n - cnt) + v * cnt - sm
        assert S.max() < 2 ** 53 and np.array_equal(cost[:, c], S / n)
        got = [int(m[k][c]) for k in ("count", "sum", "sumsq", "xmax")]
        assert got == [n, int(x64.sum()), int((x64 * x64).sum()), int(x64.max())]
        assert int(k0[c]) == np.flatnonzero(w.eta.astype(np.int64) * n <= x64.sum()).max()


# one wave a row up to 4,096 samples in the longest, else four
@pytest.mark.parametrize("sizes", [(4096, 1, 777), (4097, 1, 65), (63, 64, 65), (16_384, 255),
                                   (256, 257) * 400])
def test_moments_at_either_block_size(ctx, dev, sizes):
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(sum(sizes))
    parts = [rng.integers(0, 32769, n).astype(np.int32) for n in sizes]
    C = len(parts)
    off, xi = _csr(parts)
    w = Workload("moments", C, off, None, xi, np.full(C, 32768, np.int32), eta_grid(129, 32768),
                 lam_grid(2), _f32([1] * C), _f32([1] * C), 1, np.zeros(C, np.float32))
    prob = dro.Problem.from_workload(w, dev)
    print(f"[gpu] moments of {C} segments", flush=True)
    m = {k: v.cpu().numpy() for k, v in dro.class_moments(ctx, prob).items()}
    k0 = dro.bcd_init_state(ctx, prob).cpu().numpy()
    eta = w.eta.astype(np.int64)
    for c, x in enumerate(parts):
        x = x.astype(np.int64)
        assert [int(m[k][c]) for k in ("count", "sum", "sumsq", "xmax")] == \
            [len(x), x.sum(), (x * x).sum(), x.max()]
        assert k0[c] == np.flatnonzero(eta * len(x) <= x.sum()).max()


def test_merged_histogram_where_the_rows_do_not_fit(dev):
    import torch
    import paper_2607_16892_amd as dro
    # 50 segments of 82,000 samples: 250 or more rows of 68 KB beside 20 MB of
    # prefix entries are beyond the no-allocation array; dro_cost_eval counts in rows
    w = random_workload(seed=9, C=50, N=82_000, L=4000, K=7, M=5, E=2)
    with dro.Context(dev.index or 0) as c:
        prob = dro.Problem.from_workload(w, dev)
        eps = torch.from_numpy(w.eps.copy()).to(dev)
        ref = dro.dro_cost_eval(c, prob, eps)
        S = torch.empty((w.C, w.K, w.M), dtype=torch.float64, device=dev)
        W = torch.empty((w.E, w.C, w.K), dtype=torch.float64, device=dev)
        got = dro.dro_cost_eval_noalloc(c, prob, eps, S, W)
        torch.cuda.synchronize()
        assert torch.equal(got["S"], ref["S"]) and torch.equal(got["W"], ref["W"])
