"""Calls whose output is the input's own memory: the gradient written over the points it is
taken at, and harmonics of angles that are two rows of the output.  A point reads its own
input before it writes, so both give the bits that separate memory gives.  Where the lane
width does not divide the number of points, the last lane's first point here is the first of
a workgroup, whose neighbour may have written already."""
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


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("n", [257, (1 << 16) + 1, (1 << 18) + 1, (1 << 20) + 1, (1 << 20) + 2, (1 << 20) + 3])
@pytest.mark.parametrize("rec", [True, False])
def test_gradient_over_its_points(dev, dtype, n, rec):
    print("case: gradient in place, n", n, dtype, "rec" if rec else "explicit", flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    x = torch.randn((n, 3), generator=g, dtype=dtype, device=dev)
    G = torch.randn((16, n), generator=g, dtype=dtype, device=dev)
    fn = getattr(sh, ("sh_eval_grad_rec" if rec else "sh_eval_grad") + ("" if dtype == torch.float64 else "_f32"))
    want = fn(3, x, G)
    assert fn(3, x, G, grad_xyz=x).data_ptr() == x.data_ptr()
    assert torch.equal(x, want)


@pytest.mark.parametrize("dtype", DTYPES)
@pytest.mark.parametrize("more", [0, 1, 2, 3])
def test_harmonics_over_their_angles(dev, dtype, more):
    elem = torch.finfo(dtype).bits // 8
    n = -(-(1 << 28) // (16 * elem)) // 1024 * 1024 + 1024 + more  # lmax 3, above 2^28 bytes of output
    print("case: angles in place, n", n, dtype, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    a = torch.rand((2, n), generator=g, dtype=torch.float64, device=dev).mul_(3.1).to(dtype)
    fn = sh.sh_eval_angles if dtype == torch.float64 else sh.sh_eval_angles_f32
    want = fn(3, a[0], a[1])
    out = torch.empty((16, n), dtype=dtype, device=dev)
    out[5], out[11] = a[0], a[1]
    fn(3, out[5], out[11], out=out)
    assert torch.equal(out, want)
