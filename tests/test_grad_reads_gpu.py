"""The backward kernels' ways of reading the upstream gradient, chosen from its bytes and the
alignment of its rows (kept lines, non-temporal, kept lines off the lines): a point's
gradient is the same bits whichever is taken, around 3 x 2^26 and 2^29 bytes."""
from __future__ import annotations

import pytest
import torch

import paper_2510_05282_amd as sh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32])
@pytest.mark.parametrize("lmax", [0, 2, 3, 9, 16])
@pytest.mark.parametrize("size", [3 << 26, 1 << 29])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_reads_agree(dev, dtype, lmax, size, more):
    F, elem = (lmax + 1) ** 2, torch.finfo(dtype).bits // 8
    n = -(-size // (F * elem)) // 64 * 64 + 64 + more * (65 if more < 0 else 1)  # rows on lines for more = 0
    print("case: backward reads, lmax", lmax, "n", n, dtype, flush=True)
    g = torch.Generator(device=dev)
    g.manual_seed(n)
    x = torch.randn((n, 3), generator=g, dtype=dtype, device=dev)
    x[n // 2] = 0.0
    G = torch.randn((F, n), generator=g, dtype=dtype, device=dev)
    name = ("sh_eval_grad_rec" if lmax > 9 else "sh_eval_grad") + ("" if dtype == torch.float64 else "_f32")
    fn = getattr(sh, name)
    out = fn(lmax, x, G)
    m = n // 5 + 3
    for i in range(0, n, m):
        assert torch.equal(out[i:i + m], fn(lmax, x[i:i + m].contiguous(), G[:, i:i + m].contiguous()))


@pytest.mark.parametrize("dtype,lmax,size", [(torch.float64, 0, 3 << 24), (torch.float64, 1, 11 << 23),
                                             (torch.float64, 2, 3 << 25), (torch.float32, 2, 15 << 23),
                                             (torch.float64, 3, 15 << 23), (torch.float64, 4, 1 << 27),
                                             (torch.float32, 9, 1 << 27)])
@pytest.mark.parametrize("more", [-1, 0, 1])
def test_reads_agree_by_lmax(dev, dtype, lmax, size, more):
    """Around the sizes from which G is read past the caches."""
    test_reads_agree(dev, dtype, lmax, size, more)
