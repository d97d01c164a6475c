"""Accuracy of arithmetic that the FP32 kernels share, on the CPU: the kernels' own headers are
compiled for the host (with fused multiply-adds, as on the GPU) and their results compared with
64-bit values.  The operators' tests sum many such values, whose own rounding hides these."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

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
