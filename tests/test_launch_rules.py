"""The rules that choose a launch from sizes and alignment, on the CPU: each line below was
measured on both sides (the figures stand beside the rules), and a launch that once crossed
it was slower."""
from __future__ import annotations

import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    so = str(tmp_path_factory.mktemp("rules") / "launch_rules.so")
    subprocess.check_call([hipcc, "-x", "hip", "--cuda-host-only", "-O1", "-std=c++17", "-fPIC", "-shared",
                           os.path.join(ROOT, "tests", "host", "launch_rules.hip"), "-o", so],
                          stderr=subprocess.DEVNULL)
    L = ctypes.CDLL(so)
    L.rule_proj_lds.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int]
    return L


@pytest.mark.parametrize("f64,lmax,atoms,points,group", [
    (0, 1, 64, 17187, 0), (0, 1, 8, 137500, 0), (0, 1, 8, 300000, 0), (0, 0, 64, 25000, 0), (0, 1, 64, 62500, 1),
    (0, 1, 64, 150000, 32), (0, 1, 128, 8593, 1), (0, 1, 128, 18750, 1), (0, 0, 128, 18750, 1), (0, 2, 128, 8593, 1), (0, 2, 64, 150000, 32),
    (0, 3, 300, 3666, 1), (0, 4, 300, 3666, 1), (0, 4, 128, 8593, 1), (0, 3, 128, 31250, 32), (0, 3, 64, 150000, 0),
    (1, 0, 64, 25000, 0), (1, 0, 64, 62500, 1), (1, 0, 64, 150000, 32), (1, 0, 128, 75000, 1), (1, 1, 8, 137500, 1), (1, 1, 64, 150000, 32),
    (1, 1, 128, 75000, 1), (1, 2, 8, 1200000, 0), (1, 2, 64, 150000, 0), (1, 2, 300, 3666, 1), (1, 3, 300, 3666, 0),
    (1, 3, 300, 5333, 32), (1, 3, 64, 150000, 0)])
def test_builds_with_tables_in_lds(rules, f64, lmax, atoms, points, group):
    assert rules.rule_proj_lds(f64, lmax, atoms, atoms * points, lmax + 1, 2000) == group


@pytest.mark.parametrize("f64,lmax,knots", [(0, 4, 4096), (1, 1, 5120), (0, 1, 5120), (0, 2, 6826), (1, 2, 3413)])
def test_tables_that_fit(rules, f64, lmax, knots):
    """A CU's 160 KiB exactly (half of them for two workgroups) are taken, a knot more is not."""
    assert rules.rule_proj_lds(f64, lmax, 200, 200 * 20000, lmax + 1, knots) > 0
    assert rules.rule_proj_lds(f64, lmax, 200, 200 * 20000, lmax + 1, knots + 1) == 0
    assert rules.rule_proj_lds(f64, lmax, 200, 200 * 20000, lmax + 2, 300) == 0  # more channels than the build's
