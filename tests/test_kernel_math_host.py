"""Accuracy of arithmetic that the FP32 kernels share, on the CPU: the kernels' own headers are
compiled for the host (with fused multiply-adds, as on the GPU) and their results compared with
64-bit values.  The operators' tests sum many such values, whose own rounding hides these."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from oracle.kaiser_bessel import default_beta, kb_kernel

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1406_0359_amd", "csrc")
HARNESS = os.path.join(ROOT, "tests", "host_harness", "kernel_math.cpp")
HIP_INCLUDE = "/opt/rocm/include"


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    gxx = shutil.which("g++")
    if gxx is None or not os.path.isdir(HIP_INCLUDE):
        pytest.skip("needs g++ and the HIP headers")
    so = str(tmp_path_factory.mktemp("kernel_math") / "kernel_math.so")
    r = subprocess.run([gxx, "-std=c++17", "-O2", "-mfma", "-ffp-contract=fast", "-shared", "-fPIC", "-w",
                        "-D__HIP_PLATFORM_AMD__", "-I" + HIP_INCLUDE, "-I" + CSRC, HARNESS, "-o", so],
                       capture_output=True, text=True, timeout=300)
    assert r.returncode == 0, r.stderr[-3000:]
    return ctypes.CDLL(so)


# radix and block length of each pass after the first
PASSES = {1024: [(8, 8), (16, 64)], 2048: [(16, 32), (4, 512)], 4096: [(8, 8), (8, 64), (8, 512)]}
# A part of a twiddle is below 1 in magnitude, so one rounding moves it by at most h = 2^-25 and,
# uniform over that, by 2 h / sqrt(12) in RMS; a complex value is sqrt(2) off as much.  A table
# entry is rounded once.  A product of two entries carries both entries' roundings and two of its
# own (the product of the imaginary parts, then the multiply-add): at most 2 + 2 = 4 of them in a
# part, and in RMS sqrt(1 + 1 + 2).
H = 2.0 ** -25 * np.sqrt(2.0)
BOUND = {1024: (H, 2 * H / np.sqrt(12.0)), 2048: (H, 2 * H / np.sqrt(12.0)), 4096: (4 * H, 4 * H / np.sqrt(12.0))}


@pytest.mark.parametrize("n", sorted(PASSES))
def test_line_twiddles(lib, n):
    """Twiddles of FP32 lines: one table entry, or at 4096 the product of two."""
    exact = np.exp(-2j * np.pi * np.arange(n) / n)
    tw = np.ascontiguousarray(exact.astype(np.complex64))
    out = np.zeros(sum((r - 1) * ns for r, ns in PASSES[n]), np.complex64)
    getattr(lib, f"line_twiddles_{n}")(tw.ctypes.data_as(ctypes.c_void_p), out.ctypes.data_as(ctypes.c_void_p))
    most, rms = BOUND[n]
    at = 0
    for radix, ns in PASSES[n]:
        got = out[at:at + (radix - 1) * ns].reshape(ns, radix - 1)
        at += got.size
        m = np.arange(ns)[:, None] * np.arange(1, radix)[None, :] * (n // (ns * radix))
        err = np.abs(got - exact[m])
        assert err.max() <= most * (1 + 1e-6), (radix, ns)
        if ns >= 64:   # enough butterflies for a mean
            assert np.sqrt((err ** 2).mean(0)).max() <= rms, (radix, ns)


def _tap_polynomials(J, degree=9):
    """Coefficients [tap][k] in x = f - 1/2 of psi(f + J/2 - 1 - tap), f in [0, 1)."""
    out = []
    for a in range(J):
        p = np.polynomial.Chebyshev.interpolate(lambda x, a=a: kb_kernel(x + 0.5 * J - 0.5 - a, J, default_beta(J)), degree,
                                                domain=[-0.5, 0.5])
        out.append(p.convert(kind=np.polynomial.Polynomial, domain=[-1, 1], window=[-1, 1]).coef)
    return np.ascontiguousarray(np.array(out, np.float32))


def _horner(c, x):
    """One Horner chain a tap in FP32: a product of two FP32 values is exact in FP64, so an FP64
    product and sum rounded to FP32 is the fused multiply-add."""
    acc = np.broadcast_to(c[:, -1].astype(np.float64), (x.size, len(c)))
    for k in range(c.shape[1] - 2, -1, -1):
        acc = (acc * x[:, None].astype(np.float64) + c[:, k]).astype(np.float32).astype(np.float64)
    return acc


@pytest.mark.parametrize("fn", ["kb_taps", "kb_tap_pairs"])
@pytest.mark.parametrize("J", [4, 5, 6, 7, 8])
def test_kernel_weights(lib, J, fn):
    """The FP32 Kaiser-Bessel weights are as close to psi as one Horner chain a tap gives them.  Half
    a percent is for a different rounding of the high terms: one more rounding there reaches a
    weight times x^4, whose mean square over |x| < 1/2 is 1/2304, against a weight's own two."""
    f = np.linspace(0, 1, 20001)[:-1].astype(np.float32)
    c, x = _tap_polynomials(J), f - np.float32(0.5)
    t = (x.astype(np.float64)[:, None] + 0.5 * J - 0.5) - np.arange(J)[None, :]
    psi = kb_kernel(t, J, default_beta(J))
    got = np.zeros((f.size, J), np.float32)
    ptr = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    getattr(lib, fn)(J, ptr(c), ptr(f), f.size, ptr(got))
    rms = lambda w: np.sqrt(((w - psi) ** 2).mean())
    assert rms(got) <= 1.005 * rms(_horner(c, x))
