"""Split-K on the tile GEMMs as the model calls launch it (exe_op_gemm_model): every tile configuration with uneven last parts,
row counts on both sides of 1024, partial sums left for the next norm, and workspaces that hold fewer parts than planned.
Every row is compared; the workspace is NaN before the call and guarded behind its end."""
import numpy as np
import pytest
import torch

import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
BF16 = wl.DTYPE_BF16
GUARD = 1024


def rnd(shape, seed, scale, dtype):
    return (torch.randn(shape, generator=torch.Generator().manual_seed(seed)) * scale).to(dtype)


_ref = {}


def reference(M, N, K):
    """A . W^T in float64 (bf16 products are exact in float)."""
    if (M, N, K) not in _ref:
        _ref.clear()
        A, W = rnd((M, K), 1, 1.0, torch.bfloat16), rnd((N, K), 2, 0.05, torch.bfloat16)
        _ref[(M, N, K)] = A, W, (A.double() @ W.double().T).numpy()
    return _ref[(M, N, K)]


def check(M, N, K, cfg, splits, mode, ws_floats, defer=False):
    """mode: 0 bf16 out with relu, 1 float residual, 2 float out"""
    A, W, raw = reference(M, N, K)
    b = rnd((N,), 3, 0.5, torch.bfloat16)
    ref, act = raw + b.double().numpy(), 0 if mode == 0 else -1
    h = rnd((M, N), 4, 1.0, torch.float32)
    out = h.to(DEV) if mode == 1 else torch.full((M, N), 7.0, dtype=torch.bfloat16 if mode == 0 else torch.float32, device=DEV)
    ws = torch.full((ws_floats + GUARD,), float("nan"), device=DEV)
    left = exe.exe_op_gemm_model(BF16, M, N, K, A.to(DEV), W.to(DEV), b.to(DEV), act, 1.0, mode, out, cfg, splits, ws,
                                 4 * ws_floats, defer)
    torch.cuda.synchronize()
    assert bool(torch.isnan(ws[ws_floats:]).all()), "written behind the workspace"
    if left:
        assert torch.equal(out.cpu(), h), "out is left alone"
        got, ref = ws[:left * M * N].view(left, M, N).double().sum(0).cpu().numpy(), raw
    else:
        got = out.double().cpu().numpy()
        ref = ref + h.double().numpy() if mode == 1 else np.maximum(ref, 0) if mode == 0 else ref
    err = np.max(np.abs(got - ref), axis=1) / np.max(np.abs(ref))
    # K float additions of products of order 0.05: far below 1e-5 of the largest; a bf16 output is rounded once, 2^-9
    assert float(err.max()) < (2.0 ** -8 if mode == 0 else 1e-5), (int(err.argmax()), float(err.max()))
    return left


# cfg 0 64x256, 1 128x256, 2 256x256, 3 64x128, 4 128x128, 5 256x128, 6 192x256; parts of 11 + 10 k-tiles, 3 x 7, 4 x 4, 3 x 7 + 6,
# 5 + 4 and 9
@pytest.mark.parametrize("cfg", range(7))
@pytest.mark.parametrize("M,N", [(130, 516), (1030, 264)])
@pytest.mark.parametrize("k_tiles,splits", [(21, 2), (21, 3), (16, 4), (27, 4), (9, 2), (9, 1)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_every_configuration_with_uneven_parts(cfg, M, N, k_tiles, splits, mode):
    check(M, N, 64 * k_tiles, cfg, splits, mode, splits * M * N)


# the forms of the large kernel that are 128 and 160 features wide (5, 8): rows and features at the edges of tiles, of waves (64
# rows; 64 and 80 features) and of the 8 features that a lane stores, depths of 4 k-tiles and more
@pytest.mark.parametrize("cfg", [5, 8])
@pytest.mark.parametrize("M,N,K,splits", [(1, 4, 256, 1), (64, 80, 256, 1), (255, 156, 320, 1), (256, 164, 576, 2), (257, 320, 1024, 3),
                                          (321, 84, 256, 1), (513, 644, 512, 2), (1500, 5120, 256, 1)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_narrow_forms_of_the_large_kernel(cfg, M, N, K, splits, mode):
    check(M, N, K, cfg, splits, mode, splits * M * N if splits > 1 else 0)


# 256 x 128 tiles on either side of the line between their two kernels: whole sums of one row tile, of two, and in parts
@pytest.mark.parametrize("M,N,K,splits,large", [(130, 260, 4096 - 64, 1, 1), (130, 260, 4096, 1, 0), (257, 132, 8192 - 64, 1, 1), (257, 132, 8192, 1, 0),
                                                (1024, 132, 14336, 1, 0), (1025, 132, 14336, 1, 1), (140, 10236, 4096, 3, 1), (140, 10240, 4096, 3, 0)])
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_both_kernels_of_256_x_128_tiles(M, N, K, splits, large, mode):
    assert exe.exe_op_gemm_model_plan(BF16, M, N, K, 5, splits)[0]["large"] == large
    check(M, N, K, 5, splits, mode, splits * M * N if splits > 1 else 0)


# the reduction: rows of one group of 4 columns, of a group more than its workgroups' threads, and others that end inside one; 2 to 8
# parts, three of which it adds at a time
@pytest.mark.parametrize("M,N", [(1, 4), (257, 4), (65, 260), (33, 1028), (70, 3076)])
@pytest.mark.parametrize("splits", range(2, 9))
@pytest.mark.parametrize("mode", [0, 1, 2])
def test_reduction_of_the_parts(M, N, splits, mode):
    check(M, N, 64 * 4 * splits, 4, splits, mode, splits * M * N)


@pytest.mark.parametrize("cfg,splits", [(1, 3), (2, 2), (6, 3), (5, 2)])
def test_partial_sums_left_for_the_next_norm(cfg, splits):
    M, N, K = 1100, 516, 64 * 21
    assert check(M, N, K, cfg, splits, 1, splits * M * N, defer=True) == splits


# room for 4, 2 and 1 of the 4 parts asked for, for a part less a float, and for none
@pytest.mark.parametrize("room,parts", [(4.0, 4), (3.99, 3), (2.5, 2), (1.0, 0), (0.0, 0)])
@pytest.mark.parametrize("cfg", [2, 6, 4])
def test_fewer_parts_where_the_workspace_is_short(cfg, room, parts):
    M, N, K = 200, 260, 64 * 24
    floats = int(room * M * N)
    assert check(M, N, K, cfg, 4, 1, floats, defer=True) == parts
    check(M, N, K, cfg, 4, 0, floats)


@pytest.mark.parametrize("M,N,K", [(1025, 1024, 8192), (1500, 512, 4096), (2049, 1028, 4096), (4096, 260, 4096), (700, 1024, 4096)])
@pytest.mark.parametrize("mode", [0, 1])
def test_as_planned(M, N, K, mode):
    """The planner's own choice: at these shapes the tiles leave most of the chip idle, and K is split."""
    left = check(M, N, K, -1, 0, 1, 8 * M * N, defer=True)
    assert left > 1, left
    check(M, N, K, -1, 0, mode, 8 * M * N)
    check(M, N, K, -1, 0, mode, 0)


@pytest.mark.parametrize("M,N,cfg", [(8193, 6152, 2), (4097, 12296, 6), (3300, 15368, 1)])
def test_outputs_stored_nontemporal(M, N, cfg):
    """bf16 outputs of 96 MB and more leave by nontemporal stores; ragged rows and features."""
    assert M * N * 2 >= 96 << 20
    check(M, N, 256, cfg, 1, 0, 0)


def test_what_it_refuses():
    A = torch.zeros((64, 1024), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((64, 64), device=DEV)

    def code(K, cfg, splits, dtype=BF16, N=64):
        with pytest.raises(exe.ExeError) as e:
            exe.exe_op_gemm_model(dtype, 64, N, K, A, A, None, -1, 1.0, 2, out, cfg, splits)
        return e.value.code
    assert code(1024, 7, 1) == code(1024, 2, 5) == code(1024, 2, 17) == code(192, 6, 1) == code(1000, 2, 1) == -2
    assert code(1024, 2, 1, wl.DTYPE_F32) == code(1024, 2, 1, N=62) == -2
    assert code(1024, 2, 0) == code(1024, -1, -1) == -1
