"""Launches of several points per lane against launches of one, by sizes that follow from the
bytes written (several from 2^27 bytes and 2^16 points on): every full call below is above
both, with every remainder, and every piece it is compared with is below 2^27 bytes, so that the
two differ; the last points, where lanes overlap, also agree with the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import paper_2510_05282_amd as sh

pytestmark = pytest.mark.gpu
DTYPES = [torch.float64, torch.float32]
WIDE = 1 << 27


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _points(n, dtype, dev):
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    x = torch.randn((n, 3), generator=g, dtype=torch.float64, device=dev)
    x[n - 2] = 0.0
    return x.to(dtype).contiguous()


def _agree(fn, x, n, per_point):
    """The call over all n points and calls over pieces of fewer than 2^27 bytes."""
    assert n * per_point >= WIDE and n > 1 << 16
    y = fn(x)
    m = min(n // 3 + 1, (WIDE - 1) // per_point)
    assert m * per_point < WIDE
    for i in range(0, n, m):
        assert torch.equal(y[..., i:i + m], fn(x[i:i + m].contiguous()))
    return y


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lmax", [2, 6, 9])
@pytest.mark.parametrize("more", [0, 1, 2, 3])
def test_real_and_unit_against_the_oracle(dev, orc, dtype, lmax, more):
    elem, F = torch.finfo(dtype).bits // 8, (lmax + 1) ** 2
    n = -(-WIDE // (F * elem)) // 32 * 32 + 32 + more
    print("case: several points per lane, real, lmax", lmax, "n", n, dtype, flush=True)
    x = _points(n, dtype, dev)
    f32 = "" if dtype == torch.float64 else "_f32"
    y = _agree(lambda v: getattr(sh, "sh_eval" + f32)(lmax, v), x, n, F * elem)
    tail = slice(n - 67, n)
    ref = orc.eval_xyz(lmax, x[tail].double().cpu().numpy())
    assert np.abs(y[:, tail].cpu().numpy().astype(np.longdouble) - ref).max() <= (1e-13 if elem == 8 else 5e-6)
    u = torch.nn.functional.normalize(x.double(), dim=1).to(dtype).contiguous()
    _agree(lambda v: getattr(sh, "sh_eval_unit" + f32)(lmax, v), u, n, F * elem)


@pytest.mark.parametrize("kind,dtype,lmax", [("jac", torch.float64, 9), ("jac", torch.float64, 7),
                                             ("spinor", torch.float32, 9), ("spinor", torch.float64, 9),
                                             ("complex", torch.float32, 9), ("complex", torch.float32, 5)])
@pytest.mark.parametrize("more", [0, 1])
def test_many_rows(dev, kind, dtype, lmax, more):
    elem, F = torch.finfo(dtype).bits // 8, (lmax + 1) ** 2
    per_point = F * elem * {"complex": 2, "spinor": 8, "jac": 4}[kind]
    n = max(-(-WIDE // per_point), (1 << 16) + 2) // 32 * 32 + 32 + more
    print("case: several points per lane,", kind, "lmax", lmax, "n", n, dtype, flush=True)
    if kind == "jac":
        def fn(v):
            return torch.cat([t.reshape(-1, v.shape[0]) for t in sh.sh_eval_jac(lmax, v)])
    else:
        name = f"sh_eval_{kind}" + ("" if dtype == torch.float64 else "_f32")

        def fn(v):
            return torch.view_as_real(getattr(sh, name)(lmax, v).reshape(-1, v.shape[0])).movedim(1, -1)
    _agree(fn, _points(n, dtype, dev), n, per_point)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lmax", [1, 3, 6])
@pytest.mark.parametrize("more", [0, 1])
def test_spinors_of_angles_and_unit_vectors(dev, dtype, lmax, more):
    per_point = (lmax + 1) ** 2 * (torch.finfo(dtype).bits // 8) * 8
    n = max(-(-WIDE // per_point), (1 << 16) + 2) // 32 * 32 + 32 + more
    print("case: several points per lane, spinors of angles, lmax", lmax, "n", n, dtype, flush=True)
    a = (_points(n, dtype, dev)[:, :2] * 1.3).contiguous()
    _agree(lambda v: torch.view_as_real(sh.sh_eval_spinor_angles(lmax, v[:, 0].contiguous(), v[:, 1].contiguous())
                                        .reshape(-1, v.shape[0])).movedim(1, -1), a, n, per_point)
    u = torch.nn.functional.normalize(_points(n, torch.float64, dev), dim=1).to(dtype).contiguous()
    _agree(lambda v: torch.view_as_real(sh.sh_eval_spinor_unit(lmax, v).reshape(-1, v.shape[0])).movedim(1, -1), u, n,
           per_point)


@pytest.mark.parametrize("dtype,lmax,n", [
    (torch.float64, 16, 65537), (torch.float64, 17, 100003), (torch.float64, 24, 65536), (torch.float64, 24, 98305),
    (torch.float64, 24, 135167), (torch.float64, 24, 135169), (torch.float64, 22, 196609), (torch.float32, 24, 131072),
    (torch.float32, 24, 131073), (torch.float32, 19, 140003), (torch.float32, 10, 262146)])
def test_recurrence_against_the_split_launch(dev, orc, dtype, lmax, n):
    """The pieces are below 2^16 points, where the m are dealt to four waves whatever is written."""
    print("case: recurrence, lmax", lmax, "n", n, dtype, flush=True)
    x = _points(n, dtype, dev)
    fn = sh.sh_eval_rec if dtype == torch.float64 else sh.sh_eval_rec_f32
    y = fn(lmax, x)
    for i in range(0, n, 30001):
        assert torch.equal(y[:, i:i + 30001], fn(lmax, x[i:i + 30001].contiguous()))
    tail = slice(n - 35, n)
    ref = orc.eval_xyz(lmax, x[tail].double().cpu().numpy())
    tol = 1e-12 if dtype == torch.float64 else max(5e-6, 1e-6 * (lmax + 1))
    assert np.abs(y[:, tail].cpu().numpy().astype(np.longdouble) - ref).max() <= tol


@pytest.mark.parametrize("kind,dtype,lmax,n", [
    ("complex", torch.float64, 24, 50001), ("complex", torch.float64, 24, 81921), ("complex", torch.float64, 20, 98305),
    ("complex", torch.float32, 18, 65537), ("complex", torch.float32, 18, 65538), ("spinor", torch.float64, 24, 20001),
    ("spinor", torch.float32, 16, 65536), ("spinor", torch.float32, 16, 65537), ("spinor", torch.float32, 11, 70003)])
def test_complex_recurrence(dev, kind, dtype, lmax, n):
    """Pieces small enough for one point per lane, four degrees at a time."""
    print("case: recurrence,", kind, "lmax", lmax, "n", n, dtype, flush=True)
    per_point = (lmax + 1) ** 2 * (torch.finfo(dtype).bits // 8) * (2 if kind == "complex" else 8)
    f = sh.sh_eval_complex_rec if kind == "complex" else sh.sh_eval_spinor_rec
    x = _points(n, dtype, dev)
    y = f(lmax, x)
    m = (WIDE - 1) // per_point
    for i in range(0, n, m):
        p = f(lmax, x[i:i + m].contiguous())
        assert torch.equal(torch.view_as_real(y[..., i:i + m].contiguous()), torch.view_as_real(p))
