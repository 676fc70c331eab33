"""The one-block-per-slice schedule of the dense evaluation at its edges, S bit
for bit against the oracle: for each of the five tile shapes (512 to 8,192 pairs)
tables of one pair less, as many and one more than whole tiles, and slices around one
and two staging buffers (16,384 samples), in problems for which the launch plan (read
from its CPU build) takes that shape; tables of one pair and of a few; class sizes
around the sixteens of a step; more unequal classes than one wave looks through at
once (64) and than a block walks (512), a class of one sample beside long ones, and
sums of one slice (stored) as well as of several (added).  The pass over the table's rows
at its edges: rows longer than its stage (2,048 multipliers), more rows than a
block takes, and more (radius, row) tasks than a block has lanes; the argmin's pass
on both sides of its two kernels' border.  W, m_star and the optimum are checked
with S.
"""
import numpy as np
import pytest

import oracle
from plan_cpu import PAIRS, dense_plan
from workloads.configs import Workload, _csr, _f32, eta_grid, lam_grid

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx(dev):
    import paper_2607_16892_amd as dro
    c = dro.Context(dev.index or 0)
    yield c
    c.close()


def _check(ctx, dev, sizes, K, M, L=32768, seg=None, E=1):
    import torch
    import paper_2607_16892_amd as dro
    rng = np.random.default_rng(K * M + len(sizes))
    parts = [np.clip(np.rint(rng.lognormal(6.0, 2.0, n)), 0, L).astype(np.int32) for n in sizes]
    off, xi = _csr(parts)
    C = len(sizes) if seg is None else len(seg)
    choice = [(8.0, 1.0), (1.0, 1.0), (2.0 ** 7, 2.0 ** -10), (0.5, 3.0)]
    w = Workload("slices", C, off, None if seg is None else np.asarray(seg, np.int32), xi,
                 np.full(C, L, np.int32), eta_grid(K, L), lam_grid(M),
                 _f32([choice[c % 4][0] for c in range(C)]),
                 _f32([choice[c % 4][1] for c in range(C)]), E, _f32(rng.uniform(0, 50, E * C)))
    print(f"[gpu] slices: {C} classes, K={K} M={M}, {off[-1]} samples", flush=True)
    prob = dro.Problem.from_workload(w, dev)
    r = dro.dro_cost_eval(ctx, prob, torch.from_numpy(w.eps).to(dev))
    torch.cuda.synchronize()
    S = oracle.S_exact(w)
    assert np.array_equal(r["S"].cpu().numpy().view(np.uint64),
                          S.to_double().reshape(C, K, M).view(np.uint64))
    W, m = oracle.W_table(w, S)
    assert np.array_equal(r["W"].cpu().numpy().view(np.uint64), W.view(np.uint64))
    assert np.array_equal(r["m_star"].cpu().numpy(), m)
    a = dro.dro_argmin_reservation(ctx, prob, torch.from_numpy(w.eps).to(dev), r["S"])
    torch.cuda.synchronize()
    k, ws = oracle.argmin(W)
    assert np.array_equal(a["k_star"].cpu().numpy(), k)
    assert np.array_equal(a["W_star"].cpu().numpy().view(np.uint64), ws.view(np.uint64))


# classes of 300 samples each, and the table: one pair less, as many, one more than tiles
@pytest.mark.parametrize("shape,C,K,M", [
    (0, 64, 983, 25), (0, 64, 768, 32), (0, 32, 10923, 3),
    (1, 32, 20479, 1), (1, 32, 640, 32), (1, 8, 10923, 3),
    (2, 32, 3413, 3), (2, 32, 320, 32), (2, 8, 565, 29),
    (3, 32, 5119, 1), (3, 32, 160, 32), (3, 4, 1229, 5),
    (4, 1, 73, 7), (4, 1, 16, 32), (4, 1, 27, 19)])
def test_every_shape_around_its_tiles(ctx, dev, shape, C, K, M):
    p = dense_plan({300: C}, K, M)
    assert p["direct"] and p["shape"] == shape and (K * M + 1) % PAIRS[shape] <= 2
    _check(ctx, dev, (300, 300), K, M, seg=[c % 2 for c in range(C)])


# one block per class and tile: a slice is the class's n samples
@pytest.mark.parametrize("n", [16_383, 16_384, 16_385, 32_769])
@pytest.mark.parametrize("shape,C,K,M", [(0, 256, 8191, 1), (1, 256, 819, 5), (2, 256, 89, 23),
                                         (3, 256, 341, 3), (4, 256, 73, 7)])
def test_every_shape_around_its_buffers(ctx, dev, shape, C, K, M, n):
    p = dense_plan({n: C}, K, M)
    assert p["direct"] and p["shape"] == shape and p["P"] == 1
    _check(ctx, dev, (n, n), K, M, seg=[c % 2 for c in range(C)])


# a long slice's sums added to another's
@pytest.mark.parametrize("shape,C,K,M", [(0, 128, 8191, 1), (1, 128, 819, 5), (2, 64, 89, 23),
                                         (3, 64, 27, 19), (4, 64, 73, 7)])
def test_every_shape_with_several_long_slices(ctx, dev, shape, C, K, M):
    n = 65_537
    p = dense_plan({n: C}, K, M)
    assert p["direct"] and p["shape"] == shape and p["P"] > 1 and n // p["P"] >= 16_384
    _check(ctx, dev, (n, n), K, M, seg=[c % 2 for c in range(C)])


@pytest.mark.parametrize("K,M", [(1, 1), (1, 511), (64, 8), (27, 19), (32, 32), (25, 41),
                                 (2047, 1), (64, 64), (17, 241), (4095, 2), (64, 128), (2731, 3)])
def test_tables_around_the_tiles(ctx, dev, K, M):
    _check(ctx, dev, (700, 1, 33), K, M)


@pytest.mark.parametrize("n", [15, 16, 17, 16_383, 16_384, 16_385, 40_000, 150_001])
def test_class_sizes_around_the_buffers(ctx, dev, n):
    _check(ctx, dev, (n,), 33, 31)
    _check(ctx, dev, (n, 5), 40, 52)


def test_more_unequal_classes_than_a_wave_holds(ctx, dev):
    rng = np.random.default_rng(3)
    sizes = [int(v) for v in rng.integers(1, 3000, 131)]
    sizes[64] = 60_000
    _check(ctx, dev, sizes, 7, 11)
    _check(ctx, dev, sizes[60:70], 20, 30, seg=[c % 10 for c in range(70)])


# more sizes than the plan lists one by one, all in one of its bins, with slice counts that
# differ by one
@pytest.mark.parametrize("lo,step,C,K,M", [(8192, 15, 65, 7, 11), (40_960, 40, 100, 64, 32)])
def test_unequal_classes_of_one_bin(ctx, dev, lo, step, C, K, M):
    sizes = [lo + i * step for i in range(C)]
    p = dense_plan({n: 1 for n in sizes}, K, M)
    assert p["direct"] and len({-(-n // p["len"]) for n in sizes}) == 2
    _check(ctx, dev, sizes, K, M)


# (walked up to 512, by the table of first slices beyond; a thread of that table's launch
# holds one class up to 1,024)
@pytest.mark.parametrize("C", [512, 513, 1024, 1025, 1500, 2049])
def test_unequal_classes_around_the_table(ctx, dev, C):
    rng = np.random.default_rng(C)
    sizes = [int(v) for v in rng.integers(1, 120, 50)]
    sizes[7], sizes[49] = 70_000, 3000
    _check(ctx, dev, sizes, 7, 11, seg=rng.permutation([c % 50 for c in range(C)]))
    if C <= 1025:
        sizes = [int(v) for v in rng.integers(1, 60, C)]
        sizes[-1] = 66_000
        _check(ctx, dev, sizes, 5, 3)


@pytest.mark.parametrize("K,M,E", [(3, 2047, 2), (3, 2048, 9), (2, 2049, 9), (2, 5000, 300),
                                   (300, 1, 7), (130, 3, 70), (700, 2, 300), (65, 32, 5)])
def test_rows_and_radii_around_the_stage(ctx, dev, K, M, E):
    _check(ctx, dev, (40, 7, 300), K, M, E=E)


# the argmin's pass over S takes a wave per row from 512 rows (of up to 512 multipliers)
# and from 4,096 rows (of 256 or more), up to 32 radii
@pytest.mark.parametrize("K,M,E", [(511, 3, 1), (512, 3, 1), (600, 511, 2), (600, 512, 33),
                                   (600, 513, 2), (4095, 255, 1), (4096, 255, 1), (4096, 256, 1),
                                   (4097, 257, 3), (4100, 300, 32), (4100, 300, 33), (4096, 600, 5)])
def test_argmin_rows_around_the_wave_kernel(ctx, dev, K, M, E):
    _check(ctx, dev, (23,), K, M, E=E)
