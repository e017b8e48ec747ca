"""Launches whose lanes take 16 bytes of points at any alignment of the output rows.

Such a launch covers the points with whole vectors, the last of which overlaps its
neighbour where the lane width does not divide n; it is chosen from the bytes it
writes.  Its values are compared bit for bit with those of small calls over pieces of
the same points (one point per lane), for n around the sizes where the choice changes
and every remainder, with padded and misaligned outputs whose padding must stay
untouched."""
from __future__ import annotations

import pytest
import torch

import paper_2510_05282_amd as sh

pytestmark = pytest.mark.gpu
DTYPES = [torch.float64, torch.float32]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


def _points(n, dtype, dev, seed=0):
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    x = torch.randn((n, 3), generator=g, dtype=torch.float64, device=dev)
    x[n // 2] = 0.0  # the origin
    x[n - 1] = torch.tensor([0.0, 0.0, -1e-9], dtype=torch.float64)
    return x.to(dtype).contiguous()


def _pieces(fn, x, piece):
    return [(i, fn(x[i:i + piece].contiguous())) for i in range(0, x.shape[0], piece)]


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("lmax", [0, 1, 2, 3, 6, 9])
@pytest.mark.parametrize("more", [-1, 0, 1, 2, 3])
def test_real_rows(dev, dtype, lmax, more):
    size, F = torch.finfo(dtype).bits // 8, (lmax + 1) ** 2
    n = -(-(1 << 27) // (F * size)) // 4 * 4 + 4 + more  # about 2^27 bytes of output
    print("case: wide rows, lmax", lmax, "n", n, dtype, flush=True)
    x = _points(n, dtype, dev)
    pad, head = 5, 1  # an odd row stride and a start off the 16-byte boundary
    buf = torch.full((F * (n + pad) + head,), -7.0, dtype=dtype, device=dev)
    out = buf[head:].view(F, n + pad)
    sh.sh_eval_ld(lmax, x, out[:, :n])
    y = (sh.sh_eval if dtype == torch.float64 else sh.sh_eval_f32)(lmax, x)
    assert torch.equal(y, out[:, :n])
    assert bool((out[:, n:] == -7.0).all()) and float(buf[0]) == -7.0
    fn = sh.sh_eval if dtype == torch.float64 else sh.sh_eval_f32
    for i, p in _pieces(lambda v: fn(lmax, v), x, n // 3 + 1):
        assert torch.equal(y[:, i:i + p.shape[1]], p)


def test_real_rows_above_the_cap_size(dev):
    """2^30 bytes and more, aligned and not, where the launch reserves LDS."""
    n = (1 << 30) // 800 + 5
    print("case: wide rows above 2^30 bytes", flush=True)
    for m in (n // 2 * 2, n // 2 * 2 + 1):
        x = _points(m, torch.float64, dev, seed=m)
        y = sh.sh_eval(9, x)
        for i, p in _pieces(lambda v: sh.sh_eval(9, v), x, 150001):
            assert torch.equal(y[:, i:i + p.shape[1]], p)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kind,lmax", [("complex", 0), ("complex", 1), ("complex", 2), ("complex", 7), ("spinor", 0),
                                       ("spinor", 1), ("spinor", 4), ("jac", 0), ("jac", 1), ("jac", 5)])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_other_rows(dev, dtype, kind, lmax, more):
    if kind == "jac" and dtype == torch.float32:
        pytest.skip("the Jacobian is FP64 only")
    size, F = torch.finfo(dtype).bits // 8, (lmax + 1) ** 2
    per_point = F * size * {"complex": 2, "spinor": 8, "jac": 4}[kind]
    n = -(-(1 << 27) // per_point) // 2 * 2 + 2 + more  # about 2^27 bytes of output
    print("case: wide rows,", kind, "lmax", lmax, "n", n, dtype, flush=True)
    x = _points(n, dtype, dev)
    if kind == "jac":
        def fn(v):
            return torch.cat([t.reshape(-1, v.shape[0]) for t in sh.sh_eval_jac(lmax, v)])
    else:
        name = f"sh_eval_{kind}" + ("" if dtype == torch.float64 else "_f32")

        def fn(v):
            return torch.view_as_real(getattr(sh, name)(lmax, v).reshape(-1, v.shape[0])).movedim(1, -1)
    y = fn(x)
    for i, p in _pieces(fn, x, n // 3 + 1):
        assert torch.equal(y[..., i:i + p.shape[-1]], p)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("kind,lmax", [("real", 1), ("real", 2), ("real", 6), ("real", 7), ("complex", 1), ("complex", 3)])
@pytest.mark.parametrize("more", [0, 1])
def test_angle_rows(dev, dtype, kind, lmax, more):
    per_point = (lmax + 1) ** 2 * (torch.finfo(dtype).bits // 8) * (1 if kind == "real" else 2)
    n = -(-(1 << 27) // per_point) // 4 * 4 + 4 + more  # just over 2^27 bytes of output
    print("case: wide rows of angles,", kind, "lmax", lmax, "n", n, dtype, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    a = torch.rand((2, n), generator=g, dtype=torch.float64, device=dev).mul_(3.1).to(dtype)
    fn = {"real": sh.sh_eval_angles if dtype == torch.float64 else sh.sh_eval_angles_f32,
          "complex": sh.sh_eval_complex_angles}[kind]
    y = fn(lmax, a[0].contiguous(), a[1].contiguous())
    m = n // 3 + 1
    for i in range(0, n, m):
        p = fn(lmax, a[0, i:i + m].contiguous(), a[1, i:i + m].contiguous())
        assert torch.equal(torch.view_as_real(y[:, i:i + m]) if kind == "complex" else y[:, i:i + m],
                           torch.view_as_real(p) if kind == "complex" else p)
