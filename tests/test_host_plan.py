"""The host plans (split counts, workspace) of the built library, CPU only."""
import ctypes
import math
import os
import random
import shutil
import subprocess
from types import SimpleNamespace

import pytest

import paper_2605_31105_amd as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_2605_31105_amd")
FIELDS = ("S1", "chunk1", "S2", "chunk2", "S3", "chunk3", "csplit", "mp", "update_slots", "total",
          "S_full", "S4", "S4r")


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    if shutil.which("g++") is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("g++ or the HIP headers missing")
    G.lib()
    so = str(tmp_path_factory.mktemp("probe") / "plan_probe.so")
    subprocess.run(["g++", "-shared", "-fPIC", "-O1", "-std=c++17", "-w", "-D__HIP_PLATFORM_AMD__",
                    "-I" + os.path.join(rocm, "include"), "-I" + os.path.join(ROOT, "include"),
                    "-I" + os.path.join(PKG, "csrc"), os.path.join(ROOT, "tests", "plan_probe.cpp"),
                    G.lib_path(), "-Wl,-rpath," + PKG, "-o", so], check=True)
    fn = ctypes.CDLL(so).plan_probe
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_int32,
                   ctypes.c_void_p]

    def probe(units, group, d, dtype, n, window, budget, ragged=0):
        prob = G.Problem(units, group, d, dtype)
        out = (ctypes.c_int64 * len(FIELDS))()
        st = fn(ctypes.byref(prob), n, window, budget, ragged, out)
        return SimpleNamespace(**dict(zip(FIELDS, out))) if st == G.GRKV_OK else None

    return probe


@pytest.mark.parametrize("rows,units,keys,splits", [
    # two blocks of up to 64 rows share a compute unit: one split per unit would
    # leave half of it idle
    (32, 90, 2500, 3), (32, 155, 3370, 2), (64, 130, 2500, 2), (64, 255, 2000, 2), (64, 48, 2000, 5),
    (64, 52, 5000, 5), (64, 60, 7900, 5), (64, 60, 2500, 4),
    # a block of 128 rows fills one: whole rounds, but long units past 128 of them
    (128, 48, 2000, 5), (128, 104, 500, 2), (128, 200, 1000, 1), (128, 129, 3500, 2),
    (128, 220, 3500, 2), (128, 256, 4000, 1), (128, 130, 1100, 2), (128, 170, 2087, 2),
    (128, 170, 1900, 1), (128, 210, 2100, 1),
])
def test_key_step_splits(plan, rows, units, keys, splits):
    for d in (64, 128):
        p = plan(units, rows // 16, d, G.GRKV_BF16, 4 * keys, 16, keys)
        assert p.mp == rows and p.S_full == splits
        assert p.S_full <= p.S4r <= p.S4


@pytest.mark.parametrize("rows,units,d,n,budget", [
    (32, 131, 128, 10976, 4962), (32, 93, 64, 14335, 6199), (64, 64, 128, 4096, 512),
    (128, 40, 128, 9000, 3000), (256, 124, 128, 580, 253), (256, 59, 128, 8028, 3698),
    (32, 400, 64, 20000, 9000), (128, 8, 128, 8192, 2048), (256, 8, 128, 8192, 1024),
])
def test_fp32_splits(plan, rows, units, d, n, budget):
    # never fewer splits than one block's share of 1024 (256 for the Gram sums)
    # gives: calls with many units keep the compute units busy
    p = plan(units, rows // 16, d, G.GRKV_F32, n, 16, budget)
    ceil = lambda a, b: -(-a // b)
    def count(length, want, least):
        want = max(1, min(want, ceil(length, least)))
        return ceil(length, ceil(ceil(length, want), 32) * 32)
    assert p.S1 >= count(n, ceil(1024, units), 512)
    assert p.S2 >= count(budget, ceil(1024, units), 128) and p.chunk2 <= 8192
    assert p.S3 >= count(budget, ceil(256, units), 256)


def test_fp32_splits_fit_the_fixed_scratch(plan):
    # the finest splits that fit, not all or nothing: 2048 retained keys take
    # fewer of them than 512, and neither falls back to the coarse ones
    small = plan(8, 8, 128, G.GRKV_F32, 8192, 16, 512)
    large = plan(8, 8, 128, G.GRKV_F32, 8192, 16, 2048)
    assert max(small.total, large.total) <= G.NOALLOC_SCRATCH_BYTES
    assert small.S1 == 64 and large.S1 > 16 and large.S2 > 16
    # many units of few splits each: in as few as it takes
    for units, group, d, n, window, budget in ((26, 5, 128, 49788, 18, 39), (183, 5, 128, 4210, 9, 10),
                                               (113, 8, 64, 11847, 9, 31),
                                               (18, 4, 64, 51980, 50, 217)):
        assert plan(units, group, d, G.GRKV_F32, n, window, budget).total <= G.NOALLOC_SCRATCH_BYTES
    # a call that no splits keep inside it takes the finest
    big = plan(31, 16, 64, G.GRKV_F32, 16227, 16, 6612)
    assert big.total > G.NOALLOC_SCRATCH_BYTES and big.S1 >= 32


@pytest.mark.parametrize("units,group,n,budget,uniform,ragged", [
    (8, 4, 8192, 1024, 16, 8), (23, 8, 1422, 655, 11, 6), (11, 4, 2891, 565, 9, 5),
    (64, 4, 24001, 2000, 4, 4),
])
def test_ragged_retained_splits(plan, units, group, n, budget, uniform, ragged):
    # the shorter ranges of small calls pay where a launch sums their partials,
    # which a ragged call does not have
    assert plan(units, group, 128, G.GRKV_BF16, n, 16, budget).S2 == uniform
    assert plan(units, group, 128, G.GRKV_BF16, n, 16, budget, 1).S2 == ragged


@pytest.mark.parametrize("group,dtype", [(4, G.GRKV_BF16), (8, G.GRKV_BF16), (4, G.GRKV_F32)])
def test_equal_budgets_are_the_plain_call(plan, group, dtype):
    for window in (16, 32):
        one = G.workspace_bytes(8, group, 128, dtype, 8192, window, 512)
        assert G.workspace_bytes_ragged(8, group, 128, dtype, 8192, window, [512] * 8) == one > 0


def _plain_total(units, rows, d, bf16, n, window, budget):
    """Workspace with the split counts of even ranges alone (no finer ones, no
    rounds of blocks): what any plan of the call may fall back to."""
    ceil = lambda a, b: -(-a // b)
    def count(length, want, least):
        want = max(1, min(want, ceil(length, least)))
        return ceil(length, ceil(ceil(length, want), 32) * 32)
    mp = 32
    while mp < rows:
        mp *= 2
    fast = bf16 and mp <= 128
    want = ceil(1024, units)
    S1 = count(n, want, 512)
    if fast:
        S2 = max(count(budget, ceil(256, units), 128), ceil(budget, 4096))
        S3 = S2
    else:
        S2 = max(count(budget, want if bf16 else ceil(256, units), 128 if bf16 else 256),
                 ceil(budget, 8192))
        S3 = count(budget, ceil(256, units), 256)
    U, esz, P = units, 2 if bf16 else 4, max(n - window, 1)
    comb = U if fast and S2 >= 8 else 0
    parts = [U * S1 * mp * 4, U * S1 * mp * 8, U * mp * 8, U * mp * 4, U * S1 * mp * d * 4,
             U * mp * d * 4, U * P * 4, U * P * 4, U * budget, 0 if fast else U * budget * d * esz,
             U * S2 * mp * 4, U * S2 * mp * 8, U * mp * 8, U * mp * 4, U * S2 * mp * d * 4,
             0 if fast else mp * U * budget * 4, U * mp * d * 4, U * S3 * mp * mp * 4,
             U * S2 * mp * 4 if fast else 0, comb * mp * d * 4, comb * mp * mp * 4, comb * mp * 4,
             U * mp * mp * 4, U * d * mp * 4, U * d * mp * 2, U * d * mp * 2, U * 16, U * 128]
    return sum(ceil(b, 256) * 256 for b in parts)


def test_plans_cover_their_ranges_and_fit(plan):
    # random shapes: the splits cover each range without an empty one, in whole
    # key tiles and inside the kernels' slot limits, and a call that even ranges
    # keep inside the fixed scratch is planned inside it
    rng = random.Random(5)
    log = lambda a, b: int(math.exp(rng.uniform(math.log(a), math.log(b))))
    fit = 0
    for _ in range(20000):
        units, group = log(1, 600), rng.randint(1, 8)
        window = rng.randint(1, 256 // group)
        n = window + log(1, 60000) - 1
        budget = min(n, window + log(1, 20000) - 1)
        d, bf16 = rng.choice((64, 128)), rng.random() < 0.6
        shape = (units, group, d, n, window, budget, bf16)
        p = plan(units, group, d, G.GRKV_BF16 if bf16 else G.GRKV_F32, n, window, budget,
                 int(bf16 and rng.random() < 0.3))
        for S, chunk, length in ((p.S1, p.chunk1, n), (p.S2, p.chunk2, budget),
                                 (p.S3, p.chunk3, budget)):
            assert S >= 1 and chunk % 32 == 0 and S * chunk >= length > (S - 1) * chunk, shape
        assert p.chunk2 <= (4096 if bf16 and p.mp <= 128 else 8192), shape
        assert p.update_slots % 32 == 0 and 32 <= p.update_slots <= 4096, shape
        if _plain_total(units, group * window, d, bf16, n, window, budget) <= G.NOALLOC_SCRATCH_BYTES:
            fit += 1
            assert p.total <= G.NOALLOC_SCRATCH_BYTES, shape
    assert fit > 3000
