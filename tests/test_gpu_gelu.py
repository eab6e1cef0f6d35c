"""The GELU of batched inference (one exponential, a reciprocal and a polynomial) is no less accurate than
erff and expf: its value's and its slope's largest and rms errors against FP64, over the pre-activations
of a network (normal, of unit and of three times that width) and over evenly spaced arguments."""

import ctypes
import math
import os

import pytest
import torch

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PROBE = os.path.join(ROOT, "tests", "csrc", "libgelu_probe.so")
N = 1 << 22


def _probe():
    assert os.path.exists(PROBE), "tests/csrc/libgelu_probe.so is not built (run __graft_entry__.build())"
    lib = ctypes.CDLL(PROBE)
    lib.gelu_probe.argtypes = [ctypes.c_int, ctypes.c_int64] + [ctypes.c_void_p] * 4
    lib.gelu_probe.restype = ctypes.c_int
    return lib


def _run(lib, fast, x):
    a, d = torch.empty_like(x), torch.empty_like(x)
    stream = torch.cuda.current_stream().cuda_stream
    assert lib.gelu_probe(fast, x.numel(), x.data_ptr(), a.data_ptr(), d.data_ptr(), stream) == 0
    torch.cuda.synchronize()
    return a, d


@pytest.mark.parametrize("form", ["unit normal", "wide normal", "even 4", "even 14"])
def test_inference_gelu_is_as_accurate_as_erff(form):
    lib = _probe()
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    if form.endswith("normal"):
        x = torch.randn(N, generator=g, device="cuda") * (3.0 if form == "wide normal" else 1.0)
    else:
        half = float(form.split()[1])
        x = torch.linspace(-half, half, N, dtype=torch.float64, device="cuda").float()
    z = x.double()
    phi = 0.5 * torch.erfc(-z * math.sqrt(0.5))
    exact = (z * phi, phi + z * torch.exp(-0.5 * z * z) / math.sqrt(2.0 * math.pi))
    fast, slow = _run(lib, 1, x), _run(lib, 0, x)
    for what, f, s, e in zip(("value", "slope"), fast, slow, exact):
        f, s = f.double() - e, s.double() - e
        got = (f.abs().max().item(), f.square().mean().sqrt().item())
        ref = (s.abs().max().item(), s.square().mean().sqrt().item())
        print(f"{form} {what}: largest {got[0]:.2e}, rms {got[1]:.2e}; with erff {ref[0]:.2e}, {ref[1]:.2e}", flush=True)
        assert got[0] <= ref[0] and got[1] <= ref[1]


def test_inference_gelu_at_the_ends():
    lib = _probe()
    x = torch.tensor([0.0, -0.0, 15.9, 16.1, 1e10, 3e38, math.inf, -15.9, -1e10, -3e38, math.nan], device="cuda")
    a, d = _run(lib, 1, x)
    a_erf, d_erf = _run(lib, 0, x)
    assert a[:2].tolist() == [0.0, 0.0] and d[:2].tolist() == [0.5, 0.5]
    assert torch.equal(a[2:7], x[2:7]) and torch.all(d[2:6] == 1.0)
    assert torch.all(a[7:10] == 0.0) and torch.all(d[7:10] == 0.0)
    for i in (6, 10):  # infinite or not a number: as with erff and expf
        assert torch.equal(a[i:i + 1].nan_to_num(7.0), a_erf[i:i + 1].nan_to_num(7.0))
        assert torch.equal(d[i:i + 1].nan_to_num(7.0), d_erf[i:i + 1].nan_to_num(7.0))
