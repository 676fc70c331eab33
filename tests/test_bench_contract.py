"""The benchmark's contract, checked on the CPU."""
import os
import shutil
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
sys.path.insert(0, ROOT)

import bench  # noqa: E402


def test_dense_counters_describe_the_current_kernel():
    # The hardware-counter figures the bench line reports (VALU instructions per
    # evaluation, HBM bytes per launch) were taken on one version of the dense
    # kernel and its launch plan; they must be re-taken whenever that code changes.
    assert bench.dense_code_hash() == bench.DENSE_COUNTERS["dense_code_sha256_16"]
    src = os.path.join(ROOT, bench.DENSE_COUNTERS["source"])
    with open(src) as f:
        assert bench.DENSE_COUNTERS["dense_code_sha256_16"] in f.read()


def test_more_than_one_gpu_is_refused():
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"],
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 2
    assert "one GPU" in r.stderr
    assert r.stdout == ""


@pytest.mark.parametrize("name,old,new", [
    ("plan.h", "kBlockCycles = 12000.0", "kBlockCycles = 1.0"),
    ("plan.h", "kLoop = 8.0", "kLoop = 0.0"),
    ("plan.h", "kMaxDirectSlice = 65536", "kMaxDirectSlice = 32768"),
    ("plan.h", "kSlicesPerBlock = 16", "kSlicesPerBlock = 8"),
    ("dro_internal.h", "kHalfSadSteps = 32766", "kHalfSadSteps = 16383"),
    ("fixed.h", "const int sh = e - 117;", "const int sh = e - 116;"),
    ("wave.h", "x += dpp0<0x118>(x);", ""),
    ("dense.hip", "kT = 4096;", "kT = 2048;")])
def test_dense_code_hash_covers_kernels_and_plan(tmp_path, name, old, new):
    csrc = os.path.join(ROOT, "paper_2607_16892_amd", "csrc")
    for f in os.listdir(csrc):
        shutil.copy(os.path.join(csrc, f), tmp_path)
    assert bench.dense_code_hash(str(tmp_path)) == bench.dense_code_hash()
    text = (tmp_path / name).read_text()
    assert old in text
    (tmp_path / name).write_text(text.replace(old, new) + "\n// a comment\n")
    assert bench.dense_code_hash(str(tmp_path)) != bench.dense_code_hash()
