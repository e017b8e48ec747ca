"""Large projector builds whose workgroups hold the atom's spline table in LDS: every atom's
block is the same bits as that atom built alone (one point per lane, the table read from
memory), over few and many atoms, atoms of no or few points, tables of odd length, shared
tables and tables with more channels than the build; inconsistent offsets write nothing
out of place."""
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


def _sizes(rng, n_atoms, total):
    s = rng.integers(total // n_atoms // 2, 3 * total // n_atoms // 2, size=n_atoms)
    s[:5] = [1, 2, 3, 0, 5]
    s[-1] = 1
    s[n_atoms // 2] += max(0, total - int(s.sum())) + 7  # at least `total` points, an odd remainder
    return s


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n_atoms,channels,n_r", [(9, 0, 333), (9, 10, 2000), (200, 0, 333), (300, 10, 2000)])
@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 4])
def test_blocks_match_atoms_alone(dev, dtype, n_atoms, channels, n_r, lmax):
    rng = np.random.default_rng(n_atoms + lmax)
    sizes = _sizes(rng, n_atoms, (1 << 20) + 1)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    print("case: table in LDS, atoms", n_atoms, "points", off[-1], "lmax", lmax, dtype, flush=True)
    n_tables = max(2, n_atoms // 3)
    tabs = np.stack([workloads.radial_table(rng, channels - 1 if channels else lmax, n_r, 3.0) for _ in range(n_tables)])
    rad = sh.Radial(tabs, 3.0)
    toa = torch.from_numpy(rng.integers(-1, n_tables + 1, size=n_atoms).astype(np.int32)).to(dev)  # clamped
    cen = torch.from_numpy(rng.uniform(0.0, 10.0, size=(n_atoms, 3))).to(dev, dtype)
    g = torch.Generator(device=dev)
    g.manual_seed(lmax)
    pts = torch.rand((int(off[-1]), 3), generator=g, dtype=torch.float64, device=dev) * 3.6 - 1.8
    pts = (pts + cen.double().repeat_interleave(torch.from_numpy(sizes).to(dev), 0)).to(dtype).contiguous()
    fn = sh.sh_projectors if dtype == torch.float64 else sh.sh_projectors_f32
    F = (lmax + 1) ** 2
    out = fn(lmax, cen, torch.from_numpy(off).to(dev), pts, rad, table_of_atom=toa)
    for a in list(range(9)) + [n_atoms // 2 - 1, n_atoms // 2, n_atoms // 2 + 1, n_atoms - 2, n_atoms - 1]:
        if a >= n_atoms or sizes[a] == 0:
            continue
        for i in range(off[a], off[a + 1], 100_000):  # pieces below the large builds' sizes
            j = min(i + 100_000, int(off[a + 1]))
            one = fn(lmax, cen[a:a + 1].contiguous(), torch.tensor([0, j - i], device=dev), pts[i:j].contiguous(), rad,
                     table_of_atom=toa[a:a + 1].contiguous()).view(F, j - i)
            block = out[F * off[a]:F * off[a + 1]].view(F, int(sizes[a]))
            assert torch.equal(block[:, i - off[a]:j - off[a]], one), (a, i)
    rad.close()


@pytest.mark.parametrize("dtype", DTYPES)
def test_inconsistent_offsets(dev, dtype):
    """An atom whose range runs backwards and one that ends beyond the points: their
    blocks stay as they were or hold values of points that lie in some atom's range; the
    atoms away from them are whole and nothing beyond the output is written."""
    n_atoms, per, lmax = 256, 5000, 1
    off = np.arange(n_atoms + 1, dtype=np.int64) * per
    n = int(off[-1])
    off[100] += 3 * per  # decreasing after it
    off[-1] = n + 64     # the last atom ends beyond the points
    print("case: table in LDS, inconsistent offsets", dtype, flush=True)
    rng = np.random.default_rng(3)
    rad = sh.Radial(workloads.radial_table(rng, lmax, 500, 3.0)[None], 3.0)
    toa = torch.zeros(n_atoms, dtype=torch.int32, device=dev)
    cen = torch.zeros((n_atoms, 3), dtype=dtype, device=dev)
    g = torch.Generator(device=dev)
    g.manual_seed(1)
    pts = (torch.rand((n, 3), generator=g, dtype=torch.float64, device=dev) * 3.0 - 1.5).to(dtype).contiguous()
    F = (lmax + 1) ** 2
    buf = torch.full((F * n + 4096,), -5.0, dtype=dtype, device=dev)
    fn = sh.sh_projectors if dtype == torch.float64 else sh.sh_projectors_f32
    fn(lmax, cen, torch.from_numpy(off).to(dev), pts, rad, table_of_atom=toa, out=buf[:F * n])
    assert bool((buf[F * n:] == -5.0).all())
    assert bool((buf[F * (n_atoms - 1) * per:F * n] == -5.0).all())  # the last atom is skipped
    for a in list(range(90)) + list(range(120, n_atoms - 1)):
        one = fn(lmax, cen[:1], torch.tensor([0, per], device=dev), pts[a * per:(a + 1) * per].contiguous(), rad,
                 table_of_atom=toa[:1])
        assert torch.equal(buf[F * a * per:F * (a + 1) * per], one), a
    rad.close()
