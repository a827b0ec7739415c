"""The host plans (split counts, workspace) of the built library, CPU only."""
import ctypes
import os
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
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_int32, ctypes.c_int32, ctypes.c_void_p]

    def probe(units, group, d, dtype, n, window, budget):
        prob = G.Problem(units, group, d, dtype)
        out = (ctypes.c_int64 * len(FIELDS))()
        st = fn(ctypes.byref(prob), n, window, budget, out)
        return SimpleNamespace(**dict(zip(FIELDS, out))) if st == G.GRKV_OK else None

    return probe


@pytest.mark.parametrize("rows,units,keys,splits", [
    # two blocks of up to 64 rows share a compute unit: one split per unit would
    # leave half of it idle
    (32, 90, 2500, 3), (32, 155, 3370, 2), (64, 130, 2500, 2), (64, 255, 2000, 2), (64, 48, 2000, 5),
    # a block of 128 rows fills one: whole rounds, but long units past 128 of them
    (128, 48, 2000, 5), (128, 104, 500, 2), (128, 200, 1000, 1), (128, 129, 3500, 2),
    (128, 220, 3500, 2), (128, 256, 4000, 1),
])
def test_key_step_splits(plan, rows, units, keys, splits):
    for d in (64, 128):
        p = plan(units, rows // 16, d, G.GRKV_BF16, 4 * keys, 16, keys)
        assert p.mp == rows and p.S_full == splits
        assert p.S_full <= p.S4r <= p.S4
