"""Phi, Phi^dagger and Phi^dagger Phi for every kernel width with kernels of its own and the first
runtime width, on both sides of the changes of kernel (512, where G^T G is one launch, and 1024),
against the oracle.  Tolerances as for the other operator tests: a value sums J^2 products per
visibility or cell, so rounding stays within 1e-12 (FP64) and 1e-5 (FP32) relative."""
import numpy as np
import pytest

from gpu_cases import rand_complex, rel_l2, to_np, uv_case
from oracle.nufft import Nufft

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,M,prec", [(32, 301, "fp64"), (64, 5003, "fp32"), (512, 20011, "fp32"),
                                      (1024, 30011, "fp32"), (1024, 3001, "fp64")])
@pytest.mark.parametrize("J", [2, 3, 5, 7, 9])
def test_kernel_widths(n, M, prec, J):
    from paper_1406_0359_amd import purify
    uv = uv_case(M, n, 7 * J + n, 0.2)
    op = Nufft(n, uv, J)
    plan = purify.Plan(n, uv, J=J, levels=2, precision=prec)
    x, y = rand_complex((n, n), J), rand_complex(M, J + 1)
    if prec == "fp32":
        x, y = x.astype(np.complex64), y.astype(np.complex64)
    tol = 1e-12 if prec == "fp64" else 1e-5
    assert rel_l2(to_np(plan.phi(plan.as_vec(x))), op.phi(x)) <= tol
    assert rel_l2(to_np(plan.phi_adj(plan.as_vec(y))), op.phi_adj(y)) <= tol
    assert rel_l2(to_np(plan.normal(plan.as_vec(x))), op.normal(x)) <= tol


@pytest.mark.parametrize("n,M,J", [(32, 1, 6), (64, 1025, 7), (64, 65536, 8), (64, 65537, 8), (512, 700001, 6),
                                   (1024, 1100003, 8)])
def test_adjoint_stages_values(n, M, J):
    """FP32 units of one visibility up to the most that are staged (2048) and one above, split
    tiles among them.  Uniform cover: at 300 visibilities a cell a quantum is 6e-7 of the largest
    value, a cell's 256 roundings about 4e-6 of it."""
    from paper_1406_0359_amd import purify
    uv = uv_case(M, n, M, 1.0)
    op = Nufft(n, uv, J)
    plan = purify.Plan(n, uv, J=J, levels=2, precision="fp32")
    y = rand_complex(M, 3).astype(np.complex64)
    assert rel_l2(to_np(plan.phi_adj(plan.as_vec(y))), op.phi_adj(y)) <= 1e-5


@pytest.mark.parametrize("n,M,prec", [(256, 1572864, "fp32"), (256, 1572863, "fp32"), (256, 786433, "fp64")])
def test_adjoint_sorts_many_values(n, M, prec):
    """Visibility vectors at and below 12 MiB (above it they are sorted before gridding)."""
    from paper_1406_0359_amd import purify
    uv = uv_case(M, n, M, 0.5)
    op = Nufft(n, uv, 2)
    plan = purify.Plan(n, uv, J=2, levels=2, precision=prec)
    y = rand_complex(M, 3)
    if prec == "fp32":
        y = y.astype(np.complex64)
    tol = 1e-12 if prec == "fp64" else 1e-5
    assert rel_l2(to_np(plan.phi_adj(plan.as_vec(y))), op.phi_adj(y)) <= tol


def test_fp32_lines_of_2048_and_4096():
    """Lines of 2048 points (the shortest with the two short twiddle tables) as row, column and
    stored-operator transforms of a 2048^2 image; the stored operator against the NUFFT normal
    operator at that operator's own error (1e-4)."""
    from paper_1406_0359_amd import purify
    n, M, J = 2048, 40013, 8
    uv = uv_case(M, n, 11, 0.2)
    op = Nufft(n, uv, J)
    plan = purify.Plan(n, uv, J=J, levels=2, precision="fp32")
    x, y = rand_complex((n, n), 5).astype(np.complex64), rand_complex(M, 6).astype(np.complex64)
    assert rel_l2(to_np(plan.phi(plan.as_vec(x))), op.phi(x)) <= 1e-5
    assert rel_l2(to_np(plan.phi_adj(plan.as_vec(y))), op.phi_adj(y)) <= 1e-5
    normal = op.normal(x)
    assert rel_l2(to_np(plan.normal(plan.as_vec(x))), normal) <= 1e-5
    assert rel_l2(to_np(plan.normal(plan.as_vec(x), toeplitz=True)), normal) <= 1e-4


@pytest.mark.parametrize("J", [7, 8])
def test_adjoint_fp64_many_values(J):
    """FP64 vectors past 12 MiB: sorted before gridding with seven taps, not with eight."""
    from paper_1406_0359_amd import purify
    n, M = 256, 800003
    uv = uv_case(M, n, M, 0.5)
    plan = purify.Plan(n, uv, J=J, levels=2, precision="fp64")
    y = rand_complex(M, 3)
    assert rel_l2(to_np(plan.phi_adj(plan.as_vec(y))), Nufft(n, uv, J).phi_adj(y)) <= 1e-12
