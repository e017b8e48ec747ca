"""Projector builds on either side of 2^28 bytes written, with fewer than 2^20 points: below,
one point per lane, from there on several.  Every atom's block is the same bits as that
atom built alone, over few atoms (their data held in the lanes up to lmax 4) and many, and
where every atom has the same whole number of 128-byte lines."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2510_05282_amd as sh
from paper_2510_05282_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("lmax", [6, 9])
@pytest.mark.parametrize("n_atoms", [7, 64, 65])
@pytest.mark.parametrize("more", [0, 1, "lines"])
def test_blocks_match_atoms_alone(dev, dtype, lmax, n_atoms, more):
    F, es = (lmax + 1) ** 2, 8 if dtype == torch.float64 else 4
    total = min((1 << 28) // (F * es), (1 << 20) - 2)
    if more == "lines":
        per = (total // n_atoms + 32) // 32 * 32
        sizes = np.full(n_atoms, per)
    else:
        sizes = np.full(n_atoms, total // n_atoms)
        sizes[0], sizes[1] = 1, 2 * sizes[1] - 1
        sizes[-1] += total + more - int(sizes.sum())
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(off[-1])
    print("case: widths, atoms", n_atoms, "points", n, "lmax", lmax, dtype, flush=True)
    rng = np.random.default_rng(lmax)
    rad = sh.Radial(np.stack([workloads.radial_table(rng, lmax, 300, 3.0) for _ in range(n_atoms)]), 3.0)
    cen = torch.zeros((n_atoms, 3), dtype=dtype, device=dev)
    g = torch.Generator(device=dev)
    g.manual_seed(n_atoms)
    pts = (torch.rand((n, 3), generator=g, dtype=torch.float64, device=dev) * 3.6 - 1.8).to(dtype).contiguous()
    fn = sh.sh_projectors if dtype == torch.float64 else sh.sh_projectors_f32
    out = fn(lmax, cen, torch.from_numpy(off).to(dev), pts, rad)
    for a in (0, 1, 2, n_atoms // 2, n_atoms - 1):
        m = min(int(sizes[a]), 50_000)
        for i in (off[a], off[a + 1] - m):  # the atom's first and last points, below every wide launch
            one = fn(lmax, cen[:1], torch.tensor([0, m], device=dev), pts[i:i + m].contiguous(), rad,
                     table_of_atom=torch.tensor([a], dtype=torch.int32, device=dev)).view(F, m)
            block = out[F * off[a]:F * off[a + 1]].view(F, int(sizes[a]))
            assert torch.equal(block[:, i - off[a]:i - off[a] + m], one), (a, i)
    rad.close()
