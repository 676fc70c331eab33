"""The dense evaluation's launch plan (csrc/plan.h, host arithmetic only) compiled for
the CPU, so that tests can say which kernel, tile shape and slices a problem gets on
an MI355X (256 compute units, four resident blocks of the persistent kernel each)."""
import collections
import ctypes as ct
import functools
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2607_16892_amd", "csrc")
PAIRS = [32 * 256, 32 * 128, 32 * 64, 16 * 64, 8 * 64]  # of a tile, by shape
SRC = r'''
#include "plan.h"
extern "C" void plan(int n, const long long *size, const long long *count, int C, int K, int M,
                     long long *out)
{
    auto each = [&](auto &&add) {
        for (int i = 0; i < n; ++i) add(size[i], count[i]);
    };
    const dro::DensePlan p = dro::plan_dense(each, C, K, M, 256, 4);
    const long long v[] = {p.tiles, p.P, p.direct, p.shape, p.len, p.stored, p.blocks};
    for (int i = 0; i < 7; ++i) out[i] = v[i];
}
'''


@functools.lru_cache(maxsize=1)
def _lib():
    with tempfile.TemporaryDirectory() as d:
        src, so = os.path.join(d, "plan.cpp"), os.path.join(d, "plan.so")
        with open(src, "w") as f:
            f.write(SRC)
        subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I", CSRC, src, "-o", so],
                       check=True)
        return ct.CDLL(so)


def dense_plan(sizes, K, M):
    """The plan for `sizes`, {segment size: classes}, as a dict."""
    z = sorted(sizes.items())
    out = (ct.c_longlong * 7)()
    _lib().plan(len(z), (ct.c_longlong * len(z))(*[a for a, _ in z]),
                (ct.c_longlong * len(z))(*[b for _, b in z]), sum(b for _, b in z), K, M, out)
    return dict(zip(("tiles", "P", "direct", "shape", "len", "stored", "blocks"), out))


def workload_plan(w):
    seg = range(w.C) if w.seg is None else w.seg
    return dense_plan(collections.Counter(int(w.offsets[s + 1] - w.offsets[s]) for s in seg),
                      w.K, w.M)
