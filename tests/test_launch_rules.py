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
    L.rule_store.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int]
    L.rule_rec.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int]
    L.rule_grad_read.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int]
    L.rule_grad_rec.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_long]
    L.rule_proj_lds.argtypes = [ctypes.c_int, ctypes.c_int, ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int]
    return L


@pytest.mark.parametrize("f64,lmax,atoms,points,group", [
    (0, 1, 64, 17187, 0), (0, 1, 8, 137500, 0), (0, 1, 8, 300000, 0), (0, 0, 64, 25000, 0), (0, 1, 64, 62500, 1),
    (0, 1, 64, 150000, 32), (0, 1, 128, 8593, 1), (0, 1, 128, 18750, 1), (0, 0, 128, 18750, 1), (0, 2, 128, 8593, 1),
    (0, 2, 64, 150000, 32),
    (0, 3, 300, 3666, 1), (0, 4, 300, 3666, 1), (0, 4, 128, 8593, 1), (0, 3, 128, 31250, 32), (0, 3, 64, 150000, 0),
    (1, 0, 64, 25000, 0), (1, 0, 64, 62500, 1), (1, 0, 64, 150000, 32), (1, 0, 128, 75000, 1), (1, 1, 8, 137500, 1),
    (1, 1, 64, 150000, 32),
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


ONE, WIDE = 0, 1000  # points per lane; plus the KiB reserved


@pytest.mark.parametrize("rows,f64,n,value,reads,lines,shape", [
    # the CUs hold all workgroups of a launch of one point per lane at once (Jacobian, spinor)
    (400, 1, 42368, 8, 24, 1, ONE), (400, 1, 65536, 8, 24, 1, ONE), (400, 1, 45001, 8, 24, 0, ONE),
    (400, 1, 66048, 8, 24, 1, WIDE), (324, 0, 56064, 8, 0, 1, ONE), (324, 0, 66048, 8, 0, 1, WIDE),
    # one row, at every size that fills the GPU
    (1, 0, 25_000_000, 4, 12, 1, WIDE), (1, 0, 33_249_921, 4, 12, 0, WIDE), (1, 0, 1 << 20, 4, 12, 1, ONE),
    (1, 1, 7_499_904, 8, 24, 1, WIDE),
    # on lines, what is read counts: 115 to 134 MB written at few rows
    (9, 1, 1_597_184, 8, 24, 1, WIDE + 54), (9, 1, 1_388_672, 8, 24, 1, ONE),
    (16, 0, 2_078_080, 4, 12, 1, WIDE + 54),
    (16, 1, 1_038_976, 8, 24, 1, WIDE), (25, 0, 1_329_920, 4, 12, 1, WIDE + 54), (36, 1, 461_696, 8, 24, 1, WIDE),
    (36, 1, 461_697, 8, 24, 0, ONE), (36, 1, 399_232, 8, 24, 1, ONE), (64, 1, 259_712, 8, 24, 1, ONE),
    # FP32 lmax 3 on lines keeps two workgroups per CU
    (16, 0, 2_812_416, 4, 12, 1, WIDE + 54), (16, 0, 1_171_840, 8, 0, 1, WIDE), (16, 1, 1_406_208, 8, 24, 1, WIDE),
    # off the lines, uncapped below 5 x 2^25 bytes, then one workgroup per CU
    (64, 1, 292_865, 8, 24, 0, WIDE), (16, 1, 535_169, 16, 0, 0, WIDE), (64, 1, 429_569, 8, 24, 0, WIDE + 84),
    (9, 1, 2_083_329, 8, 24, 0, WIDE + 54), (16, 1, 1_171_841, 8, 24, 0, WIDE + 84),
    (16, 0, 2_343_681, 4, 12, 0, WIDE + 54), (25, 0, 1_499_905, 4, 12, 0, WIDE),
    # large and on lines
    (16, 0, 12_499_968, 4, 12, 1, WIDE + 84), (16, 1, 5_078_016, 16, 0, 1, WIDE + 84),
    (100, 1, 999_936, 8, 24, 1, WIDE + 84), (100, 1, 499_968, 16, 0, 1, WIDE + 54),
    (25, 1, 1 << 25, 8, 24, 1, WIDE + 54),
    (4, 1, 1 << 25, 8, 24, 1, ONE + 40), (4, 0, 1 << 25, 4, 12, 1, ONE)])
def test_store_shapes(rules, rows, f64, n, value, reads, lines, shape):
    assert rules.rule_store(rows, f64, n, value, reads, lines) == shape


REAL, COMPLEX, SPINOR = 0, 1, 2
SPLIT = 2000


@pytest.mark.parametrize("kind,f64,lmax,n,lines,unroll,shape", [
    # split below 2^16 points, whatever is written
    (REAL, 1, 16, 60000, 1, 4, SPLIT), (REAL, 1, 24, 30000, 1, 4, SPLIT), (REAL, 0, 24, 65535, 0, 4, SPLIT),
    (REAL, 1, 10, 10001, 0, 4, SPLIT),
    # one point per lane while several would leave CUs idle
    (REAL, 1, 16, 65537, 0, 4, ONE), (REAL, 1, 16, 80000, 1, 4, ONE), (REAL, 1, 16, 100000, 1, 4, WIDE + 54),
    (REAL, 0, 24, 100000, 1, 4, ONE), (REAL, 0, 16, 131072, 1, 4, ONE), (REAL, 0, 20, 140001, 0, 4, WIDE + 54),
    (REAL, 0, 10, 262144, 1, 4, WIDE + 54), (REAL, 0, 12, 170001, 0, 4, ONE), (REAL, 1, 10, 120000, 1, 4, ONE),
    (REAL, 1, 16, 1_000_001, 0, 4, WIDE + 84), (REAL, 1, 16, 1_000_000, 1, 4, WIDE + 54),
    # FP64 from 23 x 2^24 bytes on
    (REAL, 1, 24, 106_001, 0, 8, ONE), (REAL, 1, 20, 131_072, 1, 8, ONE), (REAL, 1, 20, 106_001, 0, 4, WIDE + 54),
    (REAL, 1, 20, 163_840, 1, 1, WIDE + 54), (REAL, 1, 24, 188_001, 0, 1, WIDE + 54),
    (REAL, 1, 24, 204_801, 0, 4, WIDE + 54), (COMPLEX, 1, 20, 57001, 0, 8, WIDE + 54),
    (COMPLEX, 1, 24, 57001, 0, 8, WIDE + 54), (COMPLEX, 1, 24, 90001, 0, 1, WIDE + 54),
    (COMPLEX, 1, 24, 106_001, 0, 4, WIDE + 54), (COMPLEX, 1, 16, 80001, 0, 4, WIDE + 54),
    (SPINOR, 1, 24, 30001, 0, 8, WIDE + 54), (SPINOR, 1, 16, 65537, 0, 4, WIDE + 54),
    # FP32 complex and spinor: one point while the CUs hold that in one round
    (SPINOR, 0, 16, 14514, 1, 4, ONE), (SPINOR, 0, 24, 6711, 0, 4, ONE), (SPINOR, 0, 9, 65536, 1, 4, ONE),
    (COMPLEX, 0, 24, 30000, 1, 4, ONE), (COMPLEX, 0, 20, 80001, 0, 4, WIDE + 54), (COMPLEX, 0, 9, 131_073, 0, 4, ONE)])
def test_recurrence_shapes(rules, kind, f64, lmax, n, lines, unroll, shape):
    assert rules.rule_rec(kind, f64, lmax, n, lines) == 10000 * unroll + shape


@pytest.mark.parametrize("f64,lmax,n,ppl,split,unroll", [
    (1, 16, 65535, 1, 1, 8), (0, 1, 65535, 1, 1, 8), (1, 16, 65536, 2, 1, 2), (1, 1, 262143, 2, 1, 2),
    # FP64 whole: a point and a degree at a time for few rows, else two points once one leaves no lane idle
    (1, 0, 1_500_001, 1, 0, 1), (1, 1, 400_001, 1, 0, 1), (1, 3, 4_000_001, 1, 0, 1), (1, 7, 262_144, 1, 0, 1),
    (1, 8, 262_144, 1, 0, 2), (1, 9, 327_679, 1, 0, 2), (1, 9, 327_680, 2, 0, 1), (1, 16, 400_001, 2, 0, 1),
    (1, 10, 2_000_001, 2, 0, 1),
    # FP32: whole earlier, and one point, for few rows
    (0, 0, 524_287, 2, 1, 2), (0, 0, 700_001, 1, 0, 2), (0, 1, 1_048_576, 1, 0, 2), (0, 3, 4_000_001, 1, 0, 2),
    (0, 4, 1_048_575, 2, 1, 2), (0, 4, 1_048_576, 4, 0, 2), (0, 16, 800_001, 2, 1, 2), (0, 16, 2_000_001, 4, 0, 2)])
def test_recurrence_backward_shapes(rules, f64, lmax, n, ppl, split, unroll):
    assert rules.rule_grad_rec(f64, lmax, n) == 10000 * unroll + 2000 * split + ppl


CACHED, STREAM, SHARED = 0, 1, 2


@pytest.mark.parametrize("f64,lmax,mb,lines,read", [
    # MB of G; beyond these a step's other data push it out of the memory-side cache
    (1, 9, 130, 1, CACHED), (1, 9, 160, 1, STREAM), (1, 9, 195, 0, STREAM), (0, 9, 130, 0, CACHED),
    (0, 3, 160, 1, STREAM), (1, 3, 195, 1, STREAM), (1, 2, 100, 1, CACHED), (1, 2, 130, 1, STREAM),
    (0, 2, 160, 0, STREAM), (1, 1, 80, 1, CACHED), (1, 1, 100, 1, STREAM), (1, 0, 60, 1, STREAM), (1, 0, 50, 1, CACHED),
    (1, 3, 125, 1, CACHED), (0, 3, 133, 1, STREAM), (0, 2, 125, 1, CACHED), (0, 4, 133, 0, CACHED),
    (0, 1, 195, 1, CACHED), (0, 0, 195, 1, CACHED), (0, 1, 210, 1, STREAM),
    (1, 9, 530, 0, STREAM), (1, 9, 540, 0, SHARED), (1, 9, 540, 1, STREAM), (0, 3, 900, 0, SHARED),
    (1, 2, 900, 0, STREAM)])
def test_backward_reads(rules, f64, lmax, mb, lines, read):
    n = mb * 10**6 // ((lmax + 1) ** 2 * (8 if f64 else 4))
    assert rules.rule_grad_read(f64, lmax, n, lines) == read
