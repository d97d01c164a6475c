"""Psi and Psi^dagger at the edges of the tiled wavelet kernels, against the oracle: images
smaller than a tile and levels down to a length-2 axis, one, two and all wavelet bases with and
without Dirac, and the sizes on both sides of the changes of kernel (512 and 1024).  Tolerances
as for the other operator tests: 1e-12 (FP64) and 1e-5 (FP32) in relative 2-norm; a coefficient
sums at most 16 products per axis and level."""
import numpy as np
import pytest

from gpu_cases import rand_complex, rel_l2, to_np
from oracle.sara import Sara

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,mask,levels,prec", [
    (16, 0x1FF, 4, "fp64"), (16, 1 << 8, 1, "fp32"), (32, 0x002, 5, "fp64"), (32, 0x1FE, 2, "fp32"),
    (64, 0x104, 6, "fp32"), (128, 0x1FF, 3, "fp32"), (256, 0x1FF, 1, "fp64"), (256, 0x003, 4, "fp64"),
    (512, 0x1FE, 5, "fp64"), (512, 0x041, 2, "fp32"), (1024, 0x00D, 3, "fp32"), (1024, 0x0F0, 2, "fp64"),
    (4096, 0x003, 2, "fp32"),
])
def test_dictionary_edges(n, mask, levels, prec):
    from paper_1406_0359_amd import purify
    uv = np.random.default_rng(n).uniform(-3, 3, (50, 2))
    plan = purify.Plan(n, uv, dict_mask=mask, levels=levels, precision=prec)
    sa = Sara(n, mask, levels)
    x, a = rand_complex((n, n), n + mask), rand_complex((sa.q, n, n), n + levels)
    tol = 1e-12 if prec == "fp64" else 1e-5
    assert rel_l2(to_np(plan.psi_adj(plan.as_vec(x))), sa.psi_adj(x)) <= tol
    assert rel_l2(to_np(plan.psi(plan.as_vec(a))), sa.psi(a)) <= tol


@pytest.mark.parametrize("n,mask,prec", [(2048, 0x007, "fp64"), (4096, 0x004, "fp32")])
def test_dictionary_raster_tiles(n, mask, prec):
    """Short filters where image and coefficients just reach 256 MB (four blocks in FP64, two in FP32):
    the finest synthesis takes its tiles in raster order."""
    from paper_1406_0359_amd import purify
    plan = purify.Plan(n, np.random.default_rng(n).uniform(-3, 3, (50, 2)), dict_mask=mask, levels=2, precision=prec)
    sa = Sara(n, mask, 2)
    a = rand_complex((sa.q, n, n), n)
    assert rel_l2(to_np(plan.psi(plan.as_vec(a))), sa.psi(a)) <= (1e-12 if prec == "fp64" else 1e-5)
