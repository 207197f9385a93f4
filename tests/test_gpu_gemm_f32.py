"""Float products of many rows (gemm_f32_kernel): tile edges in either direction, depths of one step and more, every way of storing,
and elements that its bf16 parts cannot hold."""
import pytest
import torch

import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def product(A, W, bias=None, act=-1, alpha=1.0, out_mode=0, out=None):
    M, K = A.shape
    N = W.shape[0]
    assert exe.exe_op_gemm_plan(wl.DTYPE_F32, M, N, K)["route"] == 0              # tiles, not the streaming kernel
    out = torch.zeros((M, N), device=DEV) if out is None else out
    exe.exe_op_gemm_model(wl.DTYPE_F32, M, N, K, A, W, bias, act, alpha, out_mode, out)
    torch.cuda.synchronize()
    return out.double().cpu()


def bound(A, W, K):
    """A sum's 6 additions per 32 k, each rounded to 2^-24 of at most the sum of magnitudes, and what is left out of the products."""
    return (6 * ((K + 31) // 32) + 4) * 2.0 ** -24 * (A.double().abs() @ W.double().abs().T)


# a shape of every tile, rows and features that end inside one
TILES = {"64x64": (2300, 324, 160), "64x128": (2111, 6148, 64), "128x128": (4033, 1540, 512)}


@pytest.fixture(params=TILES)
def shape(request):
    assert exe.GEMM_CFG_NAMES[exe.exe_op_gemm_plan(wl.DTYPE_F32, *TILES[request.param])["cfg"]] == request.param
    return TILES[request.param]


# one row, one feature quad or both in the last tiles (test_edges makes 64 x 64 tiles for the most part)
@pytest.mark.parametrize("M,N,K,tile", [(8193, 1028, 64, "64x128"), (2049, 8196, 32, "64x128"), (8321, 772, 512, "128x128"), (2049, 3076, 512, "128x128")])
def test_edges_of_the_wider_tiles(M, N, K, tile):
    assert exe.GEMM_CFG_NAMES[exe.exe_op_gemm_plan(wl.DTYPE_F32, M, N, K)["cfg"]] == tile
    test_edges(M, N, K)


@pytest.mark.parametrize("M", [2049, 2111, 2175, 12289])
@pytest.mark.parametrize("N,K", [(4, 32), (60, 64), (68, 96), (132, 256), (256, 2080), (772, 256), (1028, 32)])
def test_edges(M, N, K):
    g = torch.Generator().manual_seed(M + N + K)
    A, W = torch.randn((M, K), generator=g), torch.randn((N, K), generator=g)
    got = product(A.to(DEV), W.to(DEV))
    assert bool(((got - A.double() @ W.double().T).abs() <= bound(A, W, K)).all())


@pytest.mark.parametrize("mode", ["relu", "gelu", "resid", "f32", "alpha"])
def test_stores(mode, shape):
    M, N, K = shape
    g = torch.Generator().manual_seed(5)
    A, W, b = torch.randn((M, K), generator=g), torch.randn((N, K), generator=g) * 0.1, torch.randn((N,), generator=g)
    ref, lim = A.double() @ W.double().T, bound(A, W, K) + 2.0 ** -22 * (8 + b.double().abs())
    alpha, act, out_mode, out = 1.0, -1, 0, None
    if mode == "alpha":
        alpha = 0.37
        ref = ref * float(torch.tensor(0.37))
    ref = ref + b.double()
    if mode == "relu":
        act, ref = 0, ref.relu()
    elif mode == "gelu":                                        # slope of at most 1.13
        act, ref, lim = 1, torch.nn.functional.gelu(ref), 1.2 * lim
    elif mode == "resid":
        h = torch.randn((M, N), generator=g)
        out_mode, out, ref = 1, h.to(DEV), ref + h.double()
    elif mode == "f32":
        out_mode = 2
    got = product(A.to(DEV), W.to(DEV), b.to(DEV), act, alpha, out_mode, out)
    assert bool(((got - ref).abs() <= lim).all())


def test_values(shape):
    """Infinities, NaN, elements that round to infinity in bf16, and small ones."""
    M, N, K = shape
    g = torch.Generator().manual_seed(6)
    A, W = torch.randn((M, K), generator=g), torch.randn((N, K), generator=g) * 0.01
    A[3, 5], A[70, 0], A[71, 63], A[M - 1, 7] = float("inf"), float("-inf"), float("nan"), 3.4e38
    W[9, 2] = float("inf")
    A[100:110] *= 1e-28
    A[110, :2], W[11, :2] = 3e38, 10.0                           # overflows as a sum of floats does
    got, ref = product(A.to(DEV), W.to(DEV)), A.double() @ W.double().T
    ref = torch.where(ref.abs() > 3.4028235e38, torch.sign(ref) * float("inf"), ref)
    assert torch.equal(got.isnan(), ref.isnan())
    assert torch.equal(got.isinf(), ref.isinf()) and torch.equal(got[got.isinf()], ref[ref.isinf()])
    ok = ref.isfinite()
    # tiles with sums that are not finite are computed again with an addition per product
    lim = (K + 4) * 2.0 ** -24 * (A.double().abs() @ W.double().abs().T)
    assert bool(((got - ref).abs() <= lim)[ok].all())


@pytest.mark.parametrize("e", [-109, -115, -122, -130, -140, -149])
def test_small_operands(shape, e):
    """Operands down to the smallest floats lose nothing to the parts: the ordinary relative bound, and results that are no normal
    floats rounded once."""
    M, N, K = shape
    g = torch.Generator().manual_seed(7)
    A, W = torch.randn((M, K), generator=g), torch.randn((N, K), generator=g)
    A, W = (A.double() * 2.0 ** e).float(), (W.double() * 2.0 ** (10 if e > -149 else 30)).float()
    small = A[:N] if M >= N else A.repeat(-(-N // M), 1)[:N]          # the other way round: the weights are the small ones
    large = W[:M] if N >= M else W.repeat(-(-M // N), 1)[:M]
    for a, w in ((A, W), (large.contiguous(), small.contiguous())):
        got, ref = product(a.to(DEV), w.to(DEV)), a.double() @ w.double().T
        assert bool(((got - ref).abs() <= bound(a, w, K) + 2.0 ** -150).all())


def test_small_elements_beside_large_ones(shape):
    """What a small element adds is kept where the row's large ones meet zeros."""
    M, N, K = shape
    g = torch.Generator().manual_seed(8)
    A, W = torch.randn((M, K), generator=g), torch.randn((N, K), generator=g)
    A[:, ::2] = (A[:, ::2].double() * 2.0 ** -118).float()
    W[:, 1::2] = 0.0
    got, ref = product(A.to(DEV), W.to(DEV)), A.double() @ W.double().T
    assert bool(((got - ref).abs() <= bound(A, W, K)).all())


def test_large_sums(shape):
    """Sums and elements that are floats, but not with the parts' factor."""
    M, N, K = shape
    g = torch.Generator().manual_seed(9)
    for ea, ew in ((50, 40), (110, 0), (0, 110), (60, 60), (120, -60)):
        A, W = torch.randn((M, K), generator=g) * 2.0 ** ea, torch.randn((N, K), generator=g) * 2.0 ** ew
        got, ref = product(A.to(DEV), W.to(DEV)), A.double() @ W.double().T
        # one addition per product in the float MFMAs that compute them again
        assert bool(((got - ref).abs() <= (K + 4) * 2.0 ** -24 * (A.double().abs() @ W.double().abs().T)).all()), (ea, ew)


def test_more_tiles_than_a_launch_takes():
    """2^30 rows and a few: 2^32 threads and more."""
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 180 GB")
    n, R, N, K, more = 1 << 20, 1 << 10, 4, 32, 65
    g = torch.Generator().manual_seed(10)
    block, W = torch.randn((n, K), generator=g).to(DEV), torch.randn((N, K), generator=g).to(DEV)
    one, out = torch.zeros((n, N), device=DEV), torch.zeros((n * R + more, N), device=DEV)
    A = torch.empty((n * R + more, K), device=DEV)
    A[:n * R].view(R, n, K).copy_(block)
    A[n * R:] = block[:more]
    for x, o in ((block, one), (A, out)):
        exe.exe_op_gemm(wl.DTYPE_F32, len(x), N, K, x, W, None, -1, 1.0, 0, o)
    torch.cuda.synchronize()
    ref = block.double() @ W.double().T
    assert bool(((one.double() - ref).abs() <= bound(block, W, K)).all())
    assert all(torch.equal(o, one) for o in out[:n * R].view(R, n, N)) and torch.equal(out[n * R:], one[:more])
    del A, out
    torch.cuda.empty_cache()
