"""The GELU of the products' epilogues against 64 bits, through products with the identity matrix (which are exact)."""
import numpy as np
import pytest
import torch
from scipy.special import ndtr

import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def gelu_of(x, dtype):
    rows, k = x.shape
    td = torch.float32 if dtype == wl.DTYPE_F32 else torch.bfloat16
    a, w = x.to(td).to(DEV), torch.eye(k, dtype=td, device=DEV)
    out = torch.zeros((rows, k), dtype=td, device=DEV)
    exe.exe_op_gemm_model(dtype, rows, k, k, a, w, None, 1, 1.0, 0, out)
    return x.to(td).double().numpy(), out.double().cpu().numpy()


# the kernels that have the epilogue: plain FMA (k = 40), streaming, float tiles; bf16 tiles of either kernel
@pytest.mark.parametrize("dtype,rows,k", [(wl.DTYPE_F32, 9, 40), (wl.DTYPE_F32, 9, 64), (wl.DTYPE_F32, 4099, 64), (wl.DTYPE_BF16, 9, 64),
                                          (wl.DTYPE_BF16, 1100, 64), (wl.DTYPE_BF16, 1100, 256)])
def test_gelu_values(dtype, rows, k):
    x = torch.randn((rows, k), generator=torch.Generator().manual_seed(rows + k)) * 2.5
    x[0, :14] = torch.tensor([0.0, -0.0, 1e-30, -1e-30, 0.3, -0.3, 8.9, -8.9, 13.0, -13.0, 40.0, -40.0, 1e30, -1e30])
    x, got = gelu_of(x, dtype)
    ref = x * ndtr(x)
    err = np.abs(got - ref)
    # Float, x in (-3, 0): the exponent t * R(t) is below 16 (8.6 at 3): its rounding and that of R in front of it move its power by
    # (2^-21 + 3 * 2^-23) * ln 2 at most, power and product add 2^-23 and 2^-24: 0.8 * 2^-20.  For positive x all of it enters
    # relative to Phi >= 1/2, with exponents below 1 where the two are of a size.
    # bf16: the rounding of the result on top, half a unit of 8 significant bits: 2^-8 of the value at most.
    rnd = 0.0 if dtype == wl.DTYPE_F32 else 2.0 ** -8
    assert np.all(err[x >= 0] <= (2.0 ** -22 + rnd) * np.abs(ref[x >= 0]))
    near, far = (x < 0) & (x > -3), x <= -3
    assert np.all(err[near] <= (2.0 ** -20 + rnd) * np.abs(ref[near]))
    assert np.all(err[far] <= 1e-8 + rnd * np.abs(ref[far]))


def erf_form_in_float(x):
    f = np.float32
    erf = (2 * ndtr((x.astype(f) * f(0.5 ** 0.5)).astype(np.float64) * 2 ** 0.5) - 1).astype(f)
    return f(0.5) * x.astype(f) * (f(1) + erf)


@pytest.mark.parametrize("lo,hi", [(-9, -5), (-5, -3), (-3, -2), (-2, -1.25), (-1.25, -1), (-1, -0.75), (-0.75, -0.5), (-0.5, -0.1), (-0.1, 0),
                                   (0, 0.1), (0.1, 0.5), (0.5, 0.75), (0.75, 1), (1, 1.25), (1.25, 2), (2, 5), (5, 9)])
def test_no_less_exact_than_the_erf_form_in_any_stretch(lo, hi):
    """2-norm of the error against 64 bits, beside that of 0.5 * x * (1 + erf(x / sqrt 2)) in float with an erf that is rounded once."""
    x = lo + (hi - lo) * torch.rand((4099, 64), generator=torch.Generator().manual_seed(7), dtype=torch.float64)
    x, got = gelu_of(x.float(), wl.DTYPE_F32)
    ref = x * ndtr(x)
    # 262336 errors a side: their 2-norms vary by 0.2 % from seed to seed
    assert np.linalg.norm(got - ref) <= 1.005 * np.linalg.norm(erf_form_in_float(x).astype(np.float64) - ref)


@pytest.mark.parametrize("std", [0.05, 0.1, 0.2, 0.32, 0.5, 1.0, 2.2])
def test_no_less_exact_than_the_erf_form_over_normal_inputs(std):
    x = torch.randn((4099, 64), generator=torch.Generator().manual_seed(8), dtype=torch.float64) * std
    x, got = gelu_of(x.float(), wl.DTYPE_F32)
    ref = x * ndtr(x)
    assert np.linalg.norm(got - ref) <= 1.005 * np.linalg.norm(erf_form_in_float(x).astype(np.float64) - ref)


def test_gelu_nan():
    _, got = gelu_of(torch.full((1, 40), float("nan")), wl.DTYPE_F32)
    assert np.isnan(got).all()


def test_gelu_infinities_and_zeros():
    """The product with the identity turns infinities into NaN, so each is its row's only entry and the weights its column's only row."""
    big = np.finfo(np.float32).max
    x = torch.tensor([[float("inf")], [float("-inf")], [big], [-big], [-0.0], [0.0], [-1e-40]])
    w = torch.zeros((4, 8))
    w[:, 0] = 1
    a = torch.zeros((7, 8))
    a[:, :1] = x
    out = torch.zeros((7, 4), device=DEV)
    exe.exe_op_gemm_model(wl.DTYPE_F32, 7, 4, 8, a.to(DEV), w.to(DEV), None, 1, 1.0, 0, out)
    got = out.cpu().numpy()[:, 0]
    assert got[0] == np.inf and np.isnan(got[1]) and got[2] == big and got[3] == 0 and got[4] == 0 and got[5] == 0 and abs(got[6]) <= 1e-40
