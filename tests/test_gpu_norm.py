"""Norms at the edges of the kernel's launch shapes, and the form that finishes a split-K projection into the residual stream
first (exe_op_resid_norm), against the oracle's primitives."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16


def rnd(shape, seed, scale=1.0, dtype=torch.float32):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * scale).to(dtype)


def reference(rms, x, g, b, eps, scale):
    P, e = oracle.Primitives("double"), float(np.float32(eps))
    return (P.rmsnorm(x, g.float().numpy(), e) if rms else P.layernorm(x, g.float().numpy(), b.float().numpy(), e)) * scale


def relerr(got, ref):
    return float(np.max(np.abs(got - ref)) / np.max(np.abs(ref)))


# widths on both sides of every step of the launch rule, for few rows and for many (the rule changes at 2048 rows)
@pytest.mark.parametrize("rows", [3, 2050])
@pytest.mark.parametrize("d", [8, 256, 260, 512, 516, 1024, 1028, 2048, 2052, 4096, 4100, 5120, 5124, 8192, 8196, 12288, 12292, 16384, 16392, 20480, 20484,
                               28672, 28676, 36864])
def test_norm_launch_shapes(rows, d):
    dtype, rms = (BF16, 0) if d % 512 else (F32, 1)
    td = torch.float32 if dtype == F32 else torch.bfloat16
    x, g, b = rnd((rows, d), 1, 2.0) + 0.3, (1 + rnd((d,), 2, 0.1)).to(td), rnd((d,), 3, 0.1).to(td)
    out = torch.zeros((rows, d), dtype=td, device=DEV)
    exe.exe_op_norm(dtype, rms, x.to(DEV), None, rows, d, g.to(DEV), b.to(DEV), 1e-5, 0.5, out)
    torch.cuda.synchronize()
    pick = np.unique([0, rows // 2, rows - 1])
    ref = reference(rms, x.numpy()[pick], g, b, 1e-5, 0.5)
    # float statistics and one rounding of the result: 2^-9 relative in bf16
    assert relerr(out.float().cpu().numpy()[pick], ref) < (2e-6 if dtype == F32 else 2.0 ** -8)


@pytest.mark.parametrize("dtype,rms", [(BF16, 0), (BF16, 1), (F32, 0)])
@pytest.mark.parametrize("splits", [1, 2, 3, 4, 7, 8, 16])
@pytest.mark.parametrize("d", [64, 1024, 5120, 16388])
def test_resid_norm(dtype, rms, splits, d):
    td = torch.float32 if dtype == F32 else torch.bfloat16
    rows_all, idx = 9, [8, 0, 3, 5]
    x, part = rnd((rows_all, d), 4, 2.0), rnd((splits, rows_all, d), 5, 1.0)
    g, b, bias = (1 + rnd((d,), 6, 0.1)).to(td), rnd((d,), 7, 0.1).to(td), rnd((d,), 8, 0.5).to(td)
    for row_index in (None, idx):
        n = rows_all if row_index is None else len(idx)
        bv = bias if row_index is None else None
        xd, out = x.to(DEV).clone(), torch.zeros((n, d), dtype=td, device=DEV)
        ri = None if row_index is None else torch.tensor(row_index, dtype=torch.int32, device=DEV)
        exe.exe_op_resid_norm(dtype, rms, xd, ri, n, d, part.to(DEV), splits, rows_all, None if bv is None else bv.to(DEV),
                              g.to(DEV), b.to(DEV), 1e-6, 1.0, out)
        torch.cuda.synchronize()
        pick = np.arange(rows_all) if row_index is None else np.array(idx)
        full = x.double().numpy() + part.double().numpy().sum(0) + (0 if bv is None else bv.double().numpy())
        got = xd.cpu().numpy()
        # splits + 2 float additions of values of order 1: (splits + 2) * 2^-24 of the largest
        assert relerr(got[pick], full[pick]) < (splits + 2) * 2.0 ** -24 * 2
        rest = np.setdiff1d(np.arange(rows_all), pick)
        assert np.array_equal(got[rest], x.numpy()[rest])
        ref = reference(rms, full[pick].astype(np.float32), g, b, 1e-6, 1.0)
        assert relerr(out.float().cpu().numpy(), ref) < (1e-5 if dtype == F32 else 2.0 ** -8)


def test_order_of_a_wave_s_sum():
    """A wave adds up from lane ^ 32 down to lane ^ 1 (bits of 16-bit models follow from it): opposite values half a row of 256 apart
    cancel before anything is lost beside them.  2^27 has a last place of 16, the other lanes sum to 3 to 9 each: an order that adds a
    neighbour first shifts the mean, and with it the small elements, by several per cent."""
    x = torch.rand((1, 256), generator=torch.Generator().manual_seed(3)) * 1.5 + 0.75
    x[0, :4], x[0, 128:132] = torch.tensor([2.0 ** 27, 0, 0, 0]), torch.tensor([-2.0 ** 27, 0, 0, 0])
    g, b = torch.ones(256), torch.zeros(256)
    out = torch.zeros((1, 256), device=DEV)
    exe.exe_op_norm(F32, 0, x.to(DEV), None, 1, 256, g.to(DEV), b.to(DEV), 1e-5, 1.0, out)
    small = np.r_[4:128, 132:256]
    ref = reference(0, x.numpy(), g, b, 1e-5, 1.0)[0, small]
    # float sum of 62 lanes, difference from the mean and two products: 2^-24 each of values below 2.25, relative to differences of 0.75
    assert relerr(out.cpu().numpy()[0, small], ref) < 80 * 2.0 ** -24
