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
    # Float: the exponent 1 + t * R(t) is below 8 for t < 3, one rounding (2^-22) and that of t * R's last step move 2^-exponent by
    # 2^-21 at most, the product and the power add 2^-23; for positive x all of it enters relative to 1 - Phi(-x) >= 1/2.
    # bf16: the rounding of the result on top, half a unit of 8 significant bits: 2^-8 of the value at most.
    rnd = 0.0 if dtype == wl.DTYPE_F32 else 2.0 ** -8
    assert np.all(err[x >= 0] <= (2.0 ** -22 + rnd) * np.abs(ref[x >= 0]))
    near, far = (x < 0) & (x > -3), x <= -3
    assert np.all(err[near] <= (2.0 ** -20 + rnd) * np.abs(ref[near]))
    assert np.all(err[far] <= 1e-8 + rnd * np.abs(ref[far]))


def test_gelu_nan():
    _, got = gelu_of(torch.full((1, 40), float("nan")), wl.DTYPE_F32)
    assert np.isnan(got).all()
