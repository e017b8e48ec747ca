"""Large projector builds over atoms of very uneven size, from one point to millions: atoms
with fewer points than a table load is worth go through memory, the others through tables in
LDS, and the workgroups' shares end anywhere.  Every atom's block is the same bits as that
atom built alone, and such a build takes no longer than a few times one of as many points in
even atoms (a table load for each small atom made it 14 to 66 times as long)."""
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


def _build(dev, dtype, lmax, sizes, n_tables, n_r=700):
    rng = np.random.default_rng(lmax)
    off = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    rad = sh.Radial(np.stack([workloads.radial_table(rng, lmax, n_r, 3.0) for _ in range(n_tables)]), 3.0)
    toa = torch.from_numpy(rng.integers(0, n_tables, size=len(sizes)).astype(np.int32)).to(dev)
    cen = torch.from_numpy(rng.uniform(0.0, 1.0, size=(len(sizes), 3))).to(dev, dtype)
    g = torch.Generator(device=dev)
    g.manual_seed(lmax)
    pts = (torch.rand((int(off[-1]), 3), generator=g, dtype=torch.float64, device=dev) * 3.6 - 1.3).to(dtype)
    fn = sh.sh_projectors if dtype == torch.float64 else sh.sh_projectors_f32
    offd = torch.from_numpy(off).to(dev)
    out = torch.empty((lmax + 1) ** 2 * int(off[-1]), dtype=dtype, device=dev)
    return off, rad, toa, cen, pts.contiguous(), fn, lambda: fn(lmax, cen, offd, pts, rad, table_of_atom=toa, out=out)


def _sizes(kind):
    rng = np.random.default_rng(7)
    if kind == "tiny":  # more atoms in a wave than the 64 it looks ahead over, and empty ones
        s = np.concatenate([rng.integers(0, 4, size=900), [2_100_001]])
        s = np.concatenate([s, rng.integers(1, 13, size=200)])
    elif kind == "mixed":
        s = np.concatenate([rng.integers(1, 3000, size=300), [1_000_003, 700_001, 63, 64, 65, 1, 0, 0]])
        rng.shuffle(s)
    else:  # the whole range of a workgroup in small atoms, and the largest last
        s = np.concatenate([np.full(400, 257), [300_000], np.full(130, 1030), [1_500_000]])
    return s.astype(np.int64)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kind", ["tiny", "mixed", "blocks"])
@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 4])
def test_blocks_match_atoms_alone(dev, dtype, kind, lmax):
    sizes = _sizes(kind)
    off, rad, toa, cen, pts, fn, build = _build(dev, dtype, lmax, sizes, 5)
    print("case: uneven atoms,", kind, "points", off[-1], "lmax", lmax, dtype, flush=True)
    out, F = build(), (lmax + 1) ** 2
    n_atoms = len(sizes)
    big = np.flatnonzero(sizes > 100_000)
    some = np.unique(np.concatenate([np.arange(0, n_atoms, 23), big, np.maximum(big - 1, 0), np.minimum(big + 1, n_atoms - 1),
                                     [n_atoms - 1]]))
    for a in some:
        for i in range(int(off[a]), int(off[a + 1]), 200_000):  # pieces below the large builds' sizes
            j = min(i + 200_000, int(off[a + 1]))
            one = fn(lmax, cen[a:a + 1].contiguous(), torch.tensor([0, j - i], device=dev), pts[i:j].contiguous(), rad,
                     table_of_atom=toa[a:a + 1].contiguous()).view(F, j - i)
            block = out[F * off[a]:F * off[a + 1]].view(F, int(sizes[a]))
            assert torch.equal(block[:, i - off[a]:j - off[a]], one), (a, i)
    rad.close()


@pytest.mark.parametrize("dtype,lmax", [(torch.float32, 0), (torch.float32, 2), (torch.float32, 4), (torch.float64, 1),
                                        (torch.float64, 3)])
def test_no_slower_than_a_few_even_builds(dev, dtype, lmax):
    print("case: uneven atoms, time, lmax", lmax, dtype, flush=True)
    best = []
    for sizes in (np.full(300, 10_000), np.concatenate([[2_990_000], np.full(1000, 10)])):
        _, rad, _, _, _, _, build = _build(dev, dtype, lmax, sizes, 20, n_r=2000)
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            build()
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b))
        best.append(min(times))
        rad.close()
    assert best[1] <= 5.0 * best[0], best
