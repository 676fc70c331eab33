"""The dense evaluation's launch plan (csrc/plan.h, host arithmetic), compiled for
the CPU: over sizes from one sample to millions of classes every plan keeps its
grid below 2^32 work-items and covers all samples.
"""
import math
import random

import pytest

from plan_cpu import PAIRS, dense_plan


def _check(p, sizes, K, M):
    threads = 1024 if p["direct"] else 256
    assert 0 < p["blocks"] and p["blocks"] * threads < 1 << 32
    if p["direct"]:
        assert p["tiles"] == -(-K * M // PAIRS[p["shape"]]) and 1 <= p["len"] <= 65536
        slices = {n: -(-n // p["len"]) for n in sizes}
        assert p["blocks"] == p["tiles"] * sum(slices[n] * c for n, c in sizes.items())
        assert p["stored"] == all(s == 1 for s in slices.values())
        same = len(set(slices.values())) == 1
        assert p["P"] == (next(iter(slices.values())) if same else 0)
    else:
        T = sum(sizes.values()) * p["tiles"]
        assert p["tiles"] == -(-K * M // 8192) and p["P"] >= 1
        assert p["blocks"] <= 1024 and (p["P"] == 1 or T * p["P"] < 1 << 31)


@pytest.mark.parametrize("K,M", [(50, 10), (16, 16), (1, 1), (32, 16), (64, 32)])
@pytest.mark.parametrize("C", [(1 << 22) - 1, 1 << 22, (1 << 22) + 1, (1 << 24) + 3, 1 << 21])
def test_millions_of_classes(C, K, M):
    for sizes in ({100: C}, {100: C - 1, 70_000: 1}, {1: C // 2, 60_000: C - C // 2}):
        _check(dense_plan(sizes, K, M), sizes, K, M)


def test_sizes_over_the_whole_range():
    rng = random.Random(5)

    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    for _ in range(300):
        sizes = {log(1, 1 << 26): log(1, 1 << 12) for _ in range(rng.choice([1, 1, 2, 7, 60]))}
        K, M = log(1, 32769), log(1, 65536)
        if K * M < 1 << 31:
            _check(dense_plan(sizes, K, M), sizes, K, M)


@pytest.mark.parametrize("distinct", [63, 64, 65, 200, 5000])
@pytest.mark.parametrize("K,M", [(7, 11), (64, 32), (1000, 200)])
def test_more_sizes_than_the_plan_lists(distinct, K, M):
    rng = random.Random(distinct + K)
    sizes = {}
    while len(sizes) < distinct:
        sizes[rng.choice([rng.randint(1, 40), rng.randint(1, 90_000), rng.randint(1, 300)])
              if distinct < 300 else rng.randint(1, 90_000)] = rng.randint(1, 3)
    _check(dense_plan(sizes, K, M), sizes, K, M)


@pytest.mark.parametrize("lo,width", [(1 << 10, 128), (1 << 13, 1024), (40_960, 4096), (1 << 16, 8192),
                                      (1 << 20, 131_072)])
@pytest.mark.parametrize("distinct", [65, 100, 128])
@pytest.mark.parametrize("K,M", [(7, 11), (64, 32), (200, 100)])
def test_sizes_of_one_bin(lo, width, distinct, K, M):
    # unequal sizes in one eighth of an octave: their slice counts differ
    for step in (1, width // distinct):
        sizes = {lo + i * step: 1 for i in range(distinct)}
        _check(dense_plan(sizes, K, M), sizes, K, M)


def test_equal_sizes_give_the_plan_of_their_count():
    # bins hold their largest size, so sizes of one bin plan as if all had it
    a = {1024 + i: 2 for i in range(100)}  # one bin, more sizes than are listed one by one
    p, q = dense_plan(a, 64, 32), dense_plan({1123: 200}, 64, 32)
    assert {k: p[k] for k in ("direct", "shape", "len")} == {k: q[k] for k in ("direct", "shape", "len")}
    _check(p, a, 64, 32)
