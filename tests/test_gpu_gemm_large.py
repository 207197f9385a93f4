"""The large-tile GEMM against the oracle's linear primitive, every row compared: ragged edges in rows and features for each
tile height, features that leave 8-byte output rows (N % 8 == 4) and an output that is only 8-byte aligned, the shallowest
depth it takes, and launches in which a workgroup goes from one tile to the next."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF16 = wl.DTYPE_BF16
# bf16 products are exact in float, and K <= 1024 float additions err far below 1e-5 of the largest output; a bf16 output
# adds one rounding, 2^-9 relative
TOL = {"f32": 1e-5, "resid": 1e-5, "none": 2.0 ** -8, "relu": 2.0 ** -8, "gelu": 2.0 ** -8}
# tile height -> shapes: one row beyond a tile, one short of it, N % 8 == 4, more tiles than workgroups
SHAPES = {1: [(1025, 516, 256), (1151, 1028, 320), (1100, 12296, 1024)], 6: [(1537, 5124, 256), (4000, 2052, 256)],
          2: [(1345, 8196, 256), (4099, 3076, 256), (3073, 5124, 320)]}
# K below what the large-tile kernel takes: the same tile shapes on the other tile kernel, and the narrower tile for one round
SHALLOW = {1: [(300, 50276, 192)], 2: [(4099, 3076, 64), (8193, 6148, 192), (129, 50276, 128)], 5: [(1100, 516, 128)]}
CASES = [(cfg, *s) for group in (SHAPES, SHALLOW) for cfg, shapes in group.items() for s in shapes]
_ref = {}


def rnd(shape, seed, scale, dtype):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * scale).to(dtype)


def reference(M, N, K):
    if (M, N, K) not in _ref:
        _ref.clear()                                      # one shape at a time
        A, W = rnd((M, K), 1, 1.0, torch.bfloat16), rnd((N, K), 2, 0.05, torch.bfloat16)
        _ref[(M, N, K)] = A, W, oracle.Primitives("float").linear(A.float().numpy(), W.float().numpy(), None)
    return _ref[(M, N, K)]


@pytest.mark.parametrize("cfg,M,N,K", CASES)
@pytest.mark.parametrize("mode", sorted(TOL))
def test_large_gemm_every_row(cfg, M, N, K, mode):
    if (M, N, K) != (1100, 12296, 1024):
        assert exe.exe_op_gemm_plan(BF16, M, N, K)["cfg"] == cfg
    A, W, raw = reference(M, N, K)
    b = rnd((N,), 3, 0.5, torch.bfloat16)
    ref, alpha, act, out_mode = raw.astype(np.float64) + b.float().numpy(), 1.0, -1, 0
    out = torch.zeros((M * N + 4,), dtype=torch.bfloat16, device=DEV)
    out = out[4:].view(M, N) if mode == "none" else out[:M * N].view(M, N)        # "none": 8-byte aligned only
    if mode == "f32":
        alpha, out_mode, out = 0.37, 2, torch.zeros((M, N), dtype=torch.float32, device=DEV)
        ref = raw * np.float64(np.float32(alpha)) + b.float().numpy()
    elif mode == "resid":
        h = rnd((M, N), 4, 1.0, torch.float32)
        out, out_mode, ref = h.to(DEV), 1, ref + h.numpy()
    elif mode != "none":
        act = 0 if mode == "relu" else 1
        ref = oracle.Primitives("double").act(ref, act)
    need = exe.exe_op_gemm_workspace(BF16, M, N, K)
    ws = torch.zeros((max(need // 4, 1),), dtype=torch.float32, device=DEV)
    exe.exe_op_gemm(BF16, M, N, K, A.to(DEV), W.to(DEV), b.to(DEV), act, alpha, out_mode, out, ws)
    torch.cuda.synchronize()
    err = np.max(np.abs(out.float().cpu().numpy() - ref), axis=1) / np.max(np.abs(ref))
    assert float(err.max()) < TOL[mode], (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("M,N,K", [(8193, 1028, 64), (12289, 516, 96)])
@pytest.mark.parametrize("mode", ["f32", "resid", "gelu"])
def test_float_tiles_beyond_one_round(M, N, K, mode):
    """Float tiles of 64 x 128, more of them than CUs (64 x 64 are compared in test_gpu_gemm_stream.py, all three in test_gpu_gemm_f32.py)."""
    assert exe.exe_op_gemm_plan(wl.DTYPE_F32, M, N, K)["cfg"] == 3
    A, W, b = rnd((M, K), 1, 1.0, torch.float32), rnd((N, K), 2, 0.05, torch.float32), rnd((N,), 3, 0.5, torch.float32)
    prim = oracle.Primitives("double")
    ref, act, out_mode, out = prim.linear(A.numpy(), W.numpy(), None) + b.numpy(), -1, 2, torch.zeros((M, N), device=DEV)
    if mode == "resid":
        h = rnd((M, N), 4, 1.0, torch.float32)
        ref, out_mode, out = ref + h.numpy(), 1, h.to(DEV)
    elif mode == "gelu":
        ref, act, out_mode = prim.act(ref, 1), 1, 0
    exe.exe_op_gemm(wl.DTYPE_F32, M, N, K, A.to(DEV), W.to(DEV), b.to(DEV), act, 1.0, out_mode, out)
    torch.cuda.synchronize()
    err = np.max(np.abs(out.cpu().numpy() - ref), axis=1) / np.max(np.abs(ref))
    assert float(err.max()) < 1e-5, (int(err.argmax()), float(err.max()))     # K <= 96 float additions: far below
