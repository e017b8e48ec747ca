"""The device set-up of the radial splines (one workgroup per channel, or one thread per
channel for many short ones) against the oracle's spline, through lmax 0 projectors: at
points (r, 0, 0) about a centre at the origin the value is R_0(r) / sqrt(4 pi).

Tolerance: the projector bound 1e-13 max(1, max|R|) in FP64 and 5e-6 max(1, max|R|) in
FP32 (the tables are N(0, 1) noise, so second derivatives are as large as they get).
"""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2510_05282_amd as sh

pytestmark = pytest.mark.gpu
R_MAX = 3.0


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _build(dev, dtype, tables, table, r):
    """R_0 of `table` at the radii r, from a handle of [n_tables][1][n_r] values."""
    p = torch.zeros((r.shape[0], 3), dtype=dtype, device=dev)
    p[:, 0] = torch.from_numpy(r).to(dev, dtype)
    rad = sh.Radial(tables, R_MAX)
    out = (sh.sh_projectors if dtype == torch.float64 else sh.sh_projectors_f32)(
        0, torch.zeros((1, 3), dtype=dtype, device=dev), torch.tensor([0, r.shape[0]], device=dev), p, rad,
        table_of_atom=torch.tensor([table], dtype=torch.int32, device=dev))
    res = out.cpu().numpy()
    rad.close()
    return res


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("n_tables,n_r", [(1, 2), (1, 3), (2, 9), (3, 300), (2, 2047), (1, 2048), (1, 2049),
                                          (2, 2050), (1, 4099), (1, 20000), (300, 3), (400, 4), (385, 4)])
def test_spline_setup_lengths(dev, orc, dtype, n_tables, n_r):
    print("case: spline set-up", n_tables, "x", n_r, dtype, flush=True)
    rng = np.random.default_rng(n_r + n_tables)
    tables = rng.standard_normal((n_tables, 1, n_r))
    r = np.sort(rng.uniform(0.0, R_MAX, size=4000)).astype(np.float32).astype(np.float64)
    for t in {0, n_tables - 1}:
        got = _build(dev, dtype, tables, t, r)
        y = tables[t, 0]
        # at the radius that the lookup's r / h, rounded to double, stands for: what is
        # tested is the set-up, and on 20000 knots that rounding alone moves t by 2e-12
        q = r * (1.0 / (R_MAX / (n_r - 1)))
        r_q = np.minimum(np.longdouble(R_MAX), q.astype(np.longdouble) * R_MAX / (n_r - 1))
        ref = orc.spline_eval(y, orc.spline_setup(y, R_MAX), R_MAX, r_q) / np.sqrt(4 * np.pi)
        tol = (1e-13 if dtype == torch.float64 else 5e-6) * max(1.0, float(np.abs(y).max()))
        assert np.abs(got.astype(np.longdouble) - ref).max() <= tol


@pytest.mark.parametrize("value", [np.inf, -np.inf, np.nan, 1.7e308])
@pytest.mark.parametrize("at", [0, 2, 4])
def test_spline_setup_not_finite(dev, value, at):
    """A table with a value that is not finite (or whose differences overflow) gives the
    same from a workgroup per channel (1 table) as from a thread per channel (481)."""
    print("case: spline set-up with", value, "at", at, flush=True)
    y = np.array([0.5, -1.0, 2.0, 0.25, 1.5])
    y[at] = value
    r = np.linspace(0.0, R_MAX, 257)
    one = _build(dev, torch.float64, y[None, None], 0, r)
    many = _build(dev, torch.float64, np.repeat(y[None, None], 481, axis=0), 480, r)
    assert np.array_equal(one, many, equal_nan=True)
