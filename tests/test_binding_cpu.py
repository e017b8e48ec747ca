"""The Python binding without a GPU: errors of the runtime calls that it makes itself."""
from __future__ import annotations

import os
import subprocess
import sys

import pytest

from paper_2510_05282_amd import serve
from paper_2510_05282_amd._lib import ShError


def test_release_reports_the_failing_synchronisation(monkeypatch):
    """The wait for the current stream fails (700, an illegal address): the error names that
    call and code, the ticket is kept, and the runtime's last error does not stay behind for
    the next launch's check."""
    s = serve.Server(1 << 20, simulated=True, sim_bytes_per_s=1e12)
    a = s.add_atom(0x10000, [0, 0, 0], dtype=serve.SH_F64, n=64)
    t = s.submit(a, 1)
    assert s.wait(t, 10) == serve.DONE
    real, cleared = serve.lib(), []

    class Failing:
        def __getattr__(self, name):
            return getattr(real, name)

        def hipStreamSynchronize(self, stream):
            return 700

        def hipGetLastError(self):
            cleared.append(700)
            return 700

    with monkeypatch.context() as m:
        m.setattr(serve, "lib", Failing)
        m.setattr(serve.torch.cuda, "is_initialized", lambda: True)
        m.setattr(serve.torch._C, "_cuda_getDevice", lambda: 0)
        m.setattr(serve.torch._C, "_cuda_getCurrentRawStream", lambda d: 0)
        with pytest.raises(ShError) as e:
            s.release(t)
    assert e.value.code == 2 and e.value.hip == 700 and "hipStreamSynchronize" in str(e.value)
    assert cleared == [700]
    assert s.poll(t) == serve.DONE
    s.release(t)
    assert s.poll(t) == serve.RELEASED
    s.close()


def test_import_without_gpu_support():
    """A torch built for the CPU alone: the package imports, its host parts run, and a call on a
    CPU tensor is refused as it is with any torch."""
    code = """
import torch
for name in ("_cuda_getCurrentRawStream", "_cuda_getDevice"):
    delattr(torch._C, name)
import paper_2510_05282_amd as sh
assert sh.row(3, -2) == 10
try:
    sh.sh_eval(2, torch.randn(5, 3, dtype=torch.float64))
except (TypeError, ValueError) as e:
    print("refused", type(e).__name__)
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", code], cwd=root, capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and "refused" in r.stdout, r.stderr
