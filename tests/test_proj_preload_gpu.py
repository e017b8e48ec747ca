"""Large projector builds with several points per lane: the atoms loaded into the lanes with the
points (up to 64) or searched for, and tables that fill a CU's LDS to the last byte.  Every
atom's block is the same bits as that atom built alone (one point per lane)."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2510_05282_amd as sh
from paper_2510_05282_amd import workloads

pytestmark = pytest.mark.gpu
DTYPES = [torch.float64, torch.float32]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _check(dev, dtype, lmax, sizes, n_r, atoms):
    rng = np.random.default_rng(lmax)
    n_atoms, n_tables = len(sizes), 7
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rad = sh.Radial(np.stack([workloads.radial_table(rng, lmax, n_r, 3.0) for _ in range(n_tables)]), 3.0)
    toa = torch.from_numpy(rng.integers(0, n_tables, size=n_atoms).astype(np.int32)).to(dev)
    cen = torch.from_numpy(rng.uniform(0.0, 1.0, size=(n_atoms, 3))).to(dev, dtype)
    g = torch.Generator(device=dev)
    g.manual_seed(lmax)
    pts = (torch.rand((int(off[-1]), 3), generator=g, dtype=torch.float64, device=dev) * 3.6 - 1.3).to(dtype)
    pts[int(off[-1]) // 2] = float("nan")
    pts[-1] = cen[-1]  # the last point at its atom's centre
    fn = sh.sh_projectors if dtype == torch.float64 else sh.sh_projectors_f32
    F = (lmax + 1) ** 2
    out = fn(lmax, cen, torch.from_numpy(off).to(dev), pts, rad, table_of_atom=toa)
    for a in atoms:
        a %= n_atoms
        for i in range(off[a], off[a + 1], 40_000):  # pieces below the large builds' sizes
            j = min(i + 40_000, int(off[a + 1]))
            one = fn(lmax, cen[a:a + 1].contiguous(), torch.tensor([0, j - i], device=dev), pts[i:j].contiguous(), rad,
                     table_of_atom=toa[a:a + 1].contiguous()).view(F, j - i)
            block = out[F * off[a]:F * off[a + 1]].view(F, int(sizes[a]))[:, i - off[a]:j - off[a]]
            assert torch.allclose(block, one, rtol=0.0, atol=0.0, equal_nan=True), (a, i)  # a NaN's sign is open
    rad.close()


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lmax", [3, 4])
@pytest.mark.parametrize("n_atoms", [1, 63, 64, 65])
def test_atoms_in_the_lanes(dev, dtype, lmax, n_atoms):
    total = (1 << 20) + 77
    sizes = np.full(n_atoms, total // n_atoms)
    if n_atoms > 1:
        sizes[[0, 1, 2, -2]] = [1, 0, 3, 5]  # waves over several atoms
        sizes[n_atoms // 2] += total - int(sizes.sum())
    print("case: atoms in the lanes, atoms", n_atoms, "points", sizes.sum(), "lmax", lmax, dtype, flush=True)
    mid = n_atoms // 2
    _check(dev, dtype, lmax, sizes, 700, sorted({0, 2 % n_atoms, mid, (mid + 1) % n_atoms, n_atoms - 1}))


@pytest.mark.parametrize("dtype,lmax,n_r", [(torch.float32, 4, 4096), (torch.float32, 4, 4097), (torch.float64, 2, 3413),
                                            (torch.float64, 2, 3414), (torch.float32, 1, 5120),
                                            (torch.float64, 1, 5120)])
def test_tables_that_fill_the_lds(dev, dtype, lmax, n_r):
    """160 KiB exactly (a half of it where two workgroups share a CU), and a knot more."""
    sizes = np.full(200, 5300)
    sizes[[3, 70, -1]] = [1, 130, 20011]
    print("case: tables that fill the LDS, knots", n_r, "lmax", lmax, dtype, flush=True)
    _check(dev, dtype, lmax, sizes, n_r, [0, 3, 69, 70, 71, 150, -2, -1])
