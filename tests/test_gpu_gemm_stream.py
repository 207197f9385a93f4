"""The few-row GEMM (exe_op_gemm_stream) against the oracle's linear primitive: every instantiation at ragged edges in rows
and features, depths from one unit (fewer than its waves) to many, split over workgroups and not, every row compared; and
the float tile kernel at the edges of its tiles."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16
# bf16 products are exact in float and the sums are float: K terms of magnitude <= |a||w| err by about sqrt(K) * 2^-24 of
# their root-mean-square sum, far below 1e-5 of the largest output; a bf16 result adds one rounding, 2^-9 relative
TOL = {"f32": 1e-5, "resid": 1e-5, "relu": 2.0 ** -8, "gelu": 2.0 ** -8}


def rnd(shape, seed, scale, dtype):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * scale).to(dtype)


def check(dtype, M, N, K, mode, call):
    td = torch.float32 if dtype == F32 else torch.bfloat16
    A, W, b = rnd((M, K), 1, 1.0, td), rnd((N, K), 2, 0.05, td), rnd((N,), 3, 0.5, td)
    raw = oracle.Primitives("double").linear(A.float().numpy(), W.float().numpy(), None)
    ref, alpha, act, out_mode = raw + b.float().numpy(), 1.0, -1, 2
    out = torch.zeros((M, N), dtype=torch.float32, device=DEV)
    if mode == "f32":
        alpha = 0.37
        ref = raw * np.float64(np.float32(alpha)) + b.float().numpy()
    elif mode == "resid":
        h = rnd((M, N), 4, 1.0, torch.float32)
        out, out_mode, ref = h.to(DEV), 1, ref + h.numpy()
    else:
        act, out_mode = (0, 0) if mode == "relu" else (1, 0)
        out = torch.zeros((M, N), dtype=td, device=DEV)
        ref = oracle.Primitives("double").act(ref, act)
    call(dtype, M, N, K, A.to(DEV), W.to(DEV), b.to(DEV), act, alpha, out_mode, out)
    torch.cuda.synchronize()
    err = np.max(np.abs(out.float().cpu().numpy() - ref), axis=1) / np.max(np.abs(ref))
    assert float(err.max()) < (1e-5 if dtype == F32 else TOL[mode]), (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("ma", [1, 2, 4, 6, 8])
@pytest.mark.parametrize("nt", [1, 2, 4, 5])
def test_every_instantiation(dtype, ma, nt):
    unit = 64 if dtype == BF16 else 32
    modes = ["f32", "resid", "relu", "gelu"]
    # rows: a full block, one short of it, one more than it (a second block of one row), a single row
    for i, (M, N, units) in enumerate([(ma * 8, nt * 16, 1), (ma * 8 - 1, nt * 32 + 4, 3), (ma * 8 + 1, nt * 48 - 4, 11),
                                       (1, nt * 16 + 12, 41)]):
        print(f"stream dtype={dtype} nt={nt} ma={ma} M={M} N={N} K={units * unit}", flush=True)
        check(dtype, M, N, units * unit, modes[(i + ma + nt) % 4],
              lambda *a: exe.exe_op_gemm_stream(*a, nt=nt, ma=ma, splits=1))


@pytest.mark.parametrize("M,N,K,nt,ma,splits", [(16, 260, 64 * 64, 4, 2, 4), (3, 80, 64 * 33, 5, 1, 2), (64, 128, 64 * 130, 2, 8, 8)])
def test_split_over_workgroups(M, N, K, nt, ma, splits):
    ws = torch.full((splits * M * N,), float("nan"), device=DEV)
    for mode in ("f32", "resid", "relu"):
        check(BF16, M, N, K, mode, lambda *a: exe.exe_op_gemm_stream(*a, nt=nt, ma=ma, splits=splits, workspace=ws))


@pytest.mark.parametrize("M", [1, 7, 30, 64, 200])
@pytest.mark.parametrize("N,K", [(1024, 1024), (96, 4096), (5120, 512)])
def test_planned(M, N, K):
    ws = torch.zeros(8 * M * N, device=DEV)
    check(BF16, M, N, K, "relu", lambda *a: exe.exe_op_gemm_stream(*a, workspace=ws))
    check(F32, M, N, K, "gelu", lambda *a: exe.exe_op_gemm(*a))


@pytest.mark.parametrize("M,N,K,mode", [(4097, 128, 32, "gelu"), (2500, 516, 256, "resid"), (2049, 132, 96, "f32"), (3000, 1024, 64, "relu")])
def test_float_tile_kernel(M, N, K, mode):
    p = exe.exe_op_gemm_plan(F32, M, N, K)
    assert p["route"] == 0 and p["splits"] == 1
    check(F32, M, N, K, mode, lambda *a: exe.exe_op_gemm(*a))


def test_rejections():
    A = torch.zeros((4, 128), dtype=torch.bfloat16, device=DEV)
    W = torch.zeros((64, 128), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((4, 64), device=DEV)
    for kw, code in [(dict(nt=3, ma=1), -1), (dict(nt=1, ma=1, splits=4), -2), (dict(nt=1, ma=1, splits=0), -2)]:
        with pytest.raises(exe.ExeError) as e:
            exe.exe_op_gemm_stream(BF16, 4, 64, 128, A, W, None, -1, 1.0, 2, out, **kw)
        assert e.value.code == code
