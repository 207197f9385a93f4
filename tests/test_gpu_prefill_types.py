"""Ragged prefill attention in the types and head sizes besides bf16 x 128 (tests/test_gpu_ops.py): every row of sequences at
the edges of key tiles (64) and query tiles (128), causal and not, with and without a bias table, on the MFMA kernel and on
the row kernel that takes what it does not."""
import numpy as np
import pytest
import torch

import oracle
import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16


@pytest.mark.parametrize("dtype,dh", [(BF16, 64), (F32, 64), (F32, 128)])
@pytest.mark.parametrize("causal,use_bias", [(1, 0), (0, 1), (1, 1), (0, 0)])
@pytest.mark.parametrize("generic", [-1, 0, 1])                  # the MFMA kernel, the faster for the batch, the row kernel
@pytest.mark.parametrize("H", [3, 8])
def test_every_row(dtype, dh, causal, use_bias, generic, H):
    td = torch.float32 if dtype == F32 else torch.bfloat16
    lens = [1, 16, 63, 64, 65, 129, 257] if H == 3 else [191, 33]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    T, inner, R = int(cu[-1]), H * dh, 50
    g = torch.Generator().manual_seed(100 + dh + H)
    qkv = torch.randn((T, 3 * inner), generator=g).to(td)
    tab = (torch.randn((H, 2 * R + 1), generator=g) * 0.5) if use_bias else None
    out = torch.zeros((T, inner), dtype=td, device=DEV)
    scale = 1.0 / np.sqrt(dh) if causal else 0.11
    exe.exe_op_prefill_attention(dtype, cu, qkv.to(DEV), H, dh, scale, causal, None if tab is None else tab.to(DEV), R, out,
                                 force_generic=generic)
    torch.cuda.synchronize()
    got, x = out.float().cpu().numpy(), qkv.double().numpy()
    worst = 0.0
    for s, L in enumerate(lens):
        for h in range(H):
            q, k, v = (x[cu[s]:cu[s + 1], j * inner + h * dh:j * inner + (h + 1) * dh] for j in range(3))
            sc = (q @ k.T) * float(np.float32(scale))
            i, j = np.arange(L)[:, None], np.arange(L)[None, :]
            if use_bias:
                sc += tab.double().numpy()[h][np.clip(j - i, -R, R) + R]
            if causal:
                sc = np.where(j <= i, sc, -np.inf)
            p = np.exp(sc - sc.max(axis=1, keepdims=True))
            ref = (p / p.sum(axis=1, keepdims=True)) @ v
            err = np.abs(got[cu[s]:cu[s + 1], h * dh:(h + 1) * dh] - ref).max(axis=1) / np.abs(ref).max(axis=1)
            worst = max(worst, float(err.max()))
    # float sums and probabilities throughout; in bf16 one rounding of the result, 2^-9
    assert worst < (1e-5 if dtype == F32 else 2.0 ** -8), worst


# 22 workgroups a copy: bf16 x 128 in the form of few (64 rows each, two value buffers), of some (causal only: two buffers) and of many
@pytest.mark.parametrize("dtype,dh,copies", [(BF16, 128, 1), (BF16, 128, 25), (BF16, 128, 60), (BF16, 64, 1), (F32, 64, 1), (F32, 128, 1)])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("R", [1, 31, 64, 128, 511])              # radius of the bias table: none to all of the tiles look it up
def test_bias_radius(dtype, dh, copies, causal, R):
    td = torch.float32 if dtype == F32 else torch.bfloat16
    lens, H = [1, 65, 352, 700], 2
    cu = np.concatenate([[0], np.cumsum(lens * copies)]).astype(np.int32)
    T, inner = sum(lens), H * dh
    g = torch.Generator().manual_seed(R + dh)
    qkv = torch.randn((T, 3 * inner), generator=g).to(td)
    tab = torch.randn((H, 2 * R + 1), generator=g)
    out = torch.zeros((copies * T, inner), dtype=td, device=DEV)
    exe.exe_op_prefill_attention(dtype, cu, qkv.to(DEV).repeat(copies, 1), H, dh, 0.11, causal, tab.to(DEV), R, out, force_generic=-1)
    torch.cuda.synchronize()
    out = out.reshape(copies, T, inner)
    assert all(torch.equal(out[i], out[0]) for i in range(copies))
    got, x = out[0].double().cpu(), qkv.double()
    worst = 0.0
    for s, L in enumerate(lens):
        q, k, v = (x[cu[s]:cu[s + 1], j * inner:(j + 1) * inner].reshape(L, H, dh).transpose(0, 1).contiguous() for j in range(3))
        rel = torch.arange(L)[None, :] - torch.arange(L)[:, None]
        sc = (q @ k.transpose(1, 2).contiguous()) * float(np.float32(0.11)) + tab.double()[:, rel.clamp(-R, R) + R]
        if causal:
            sc = sc.masked_fill(rel > 0, float("-inf"))
        ref = (sc.softmax(dim=-1) @ v).transpose(0, 1).reshape(L, H, dh)
        err = (got[cu[s]:cu[s + 1]].reshape(L, H, dh) - ref).abs().amax(dim=2) / ref.abs().amax(dim=2)
        worst = max(worst, float(err.max()))
    # as above; bf16 x 128 rounds its probabilities to bf16 before the second product too
    assert worst < (1e-5 if dtype == F32 else 2.0 ** -8 if dh == 64 else 2.0 ** -6), worst


@pytest.mark.parametrize("dtype,dh,copies", [(BF16, 128, (10, 25)), (BF16, 64, (25,)), (F32, 64, (10,))])
@pytest.mark.parametrize("causal,use_bias", [(1, 0), (0, 1), (1, 1), (0, 0)])
@pytest.mark.parametrize("H", [5, 8])
def test_forms_agree(dtype, dh, copies, causal, use_bias, H):
    """The kernel's form depends on how many workgroups a batch makes; a sequence's rows do not."""
    td = torch.float32 if dtype == F32 else torch.bfloat16
    lens, R = [1, 63, 64, 65, 130, 200, 300], 50
    T, inner = sum(lens), H * dh
    g = torch.Generator().manual_seed(dh + H)
    qkv = torch.randn((T, 3 * inner), generator=g).to(td).to(DEV)
    tab = (torch.randn((H, 2 * R + 1), generator=g) * 0.5).to(DEV) if use_bias else None

    def run(n, generic=-1):
        cu = np.concatenate([[0], np.cumsum(lens * n)]).astype(np.int32)
        out = torch.zeros((n * T, inner), dtype=td, device=DEV)
        exe.exe_op_prefill_attention(dtype, cu, qkv.repeat(n, 1), H, dh, 0.11, causal, tab, R, out, force_generic=generic)
        torch.cuda.synchronize()
        return out.reshape(n, T, inner)

    one, rows = run(1), run(1, 1)
    # against the row kernel: a rounding of either in bf16, and of the probabilities at head size 128; sums in float
    worst = float(((one - rows).float().abs().amax(dim=2) / rows.float().abs().amax(dim=2)).max())
    assert worst < (1e-5 if dtype == F32 else 2.0 ** -7 if dh == 64 else 2.0 ** -6), worst
    for n in copies:
        many = run(n)
        assert all(torch.equal(many[i], one[0]) for i in (0, n // 2, n - 1)), n


def float64_attention(x, H, dh, scale):
    q, k, v = (x.double()[:, j * H * dh:(j + 1) * H * dh].reshape(-1, H, dh).transpose(0, 1).contiguous() for j in range(3))
    return (((q @ k.transpose(1, 2).contiguous()) * scale).softmax(dim=-1) @ v).transpose(0, 1).reshape(-1, H, dh)


def float_rows(x, H, dh, scale):
    out = torch.zeros((len(x), H * dh), device=DEV)
    exe.exe_op_prefill_attention(F32, np.array([0, len(x)], dtype=np.int32), x.to(DEV), H, dh, scale, 0, None, 0, out, force_generic=-1)
    torch.cuda.synchronize()
    return out.double().cpu().reshape(-1, H, dh)


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("qe,ke,ve", [(0, 0, -110), (0, 0, -118), (0, 0, -126), (-118, 0, 0), (0, -122, 0), (-60, -60, -122), (-110, 110, 0),
                                      (0, 0, 90), (0, 0, 115), (40, 42, 0)])
def test_float_range(dh, qe, ke, ve):
    """Queries, keys and values of any size: as exact as ordinary ones.  The scale makes up for the scores'."""
    n, H = 200, 2
    g = torch.Generator().manual_seed(dh - qe)
    x = torch.randn((n, 3 * H * dh), generator=g).double()
    for j, e in enumerate((qe, ke, ve)):
        x[:, j * H * dh:(j + 1) * H * dh] *= 2.0 ** e
    x, scale = x.float(), float(np.float32(0.11)) * 2.0 ** -(qe + ke)
    ref, got = float64_attention(x, H, dh, scale), float_rows(x, H, dh, scale)
    err = (got - ref).abs().amax(dim=2) / ref.abs().amax(dim=2)
    assert float(err.max()) < 1e-5, float(err.max())


@pytest.mark.parametrize("dh", [64, 128])
def test_float_small_probabilities(dh):
    """A key that takes all but 2^-119 to 2^-125 of a row, with a value of zero: the row is what the others add."""
    n = 64
    x = torch.zeros((n, 3 * dh))
    # scores of key 0: 82.5 to 86.6, the others' zero (from 87.4 on exp2 gives 2^-126 and less, zero in every form of the kernel)
    x[:, 0] = 1.0 + torch.arange(n) / 1280.0
    x[0, dh] = 82.5 / 0.125
    x[1:, 2 * dh:] = torch.randn((n - 1, dh), generator=torch.Generator().manual_seed(1))
    ref, got = float64_attention(x, 1, dh, 0.125), float_rows(x, 1, dh, 0.125)
    # the exponent, 125 for exp2, is the product of three roundings: 3 * 125 * 2^-24 * ln 2, and the sums' own
    err = (got - ref).abs().amax(dim=2) / ref.abs().amax(dim=2)
    assert float(err.max()) < 2e-5, float(err.max())


@pytest.mark.parametrize("dh", [64, 128])
def test_float_scores_about_2_to_the_80(dh):
    """Scores that are floats, but not with the factor that the parts carry, beside others that are: every key counts."""
    n = 64
    x = torch.zeros((n, 3 * dh), dtype=torch.float64)
    x[:, 0] = 2.0 ** 40
    x[:, dh] = -2.0 ** 40 * (1 + (torch.arange(n) - 2) * 2.0 ** -23)              # an eighth apart with the scale: keys 0 .. 2 are above
    x[:, 2 * dh:] = torch.arange(n)[:, None]
    x = x.float()
    ref, got = float64_attention(x, 1, dh, 2.0 ** -60), float_rows(x, 1, dh, 2.0 ** -60)
    # floats of 2^20 log2(e) are an eighth apart, so an exponent is off by up to a sixteenth: a weight by 2^(1/16), a ratio by 2^(1/8)
    assert float((got / ref - 1).abs().max()) < 0.1 and float(ref.min()) > 5


def test_more_workgroups_than_a_launch_takes():
    """Half a million sequences of 2 and 3 tokens, 16 heads: 2^32 threads and more, which are no single launch."""
    n, H, dh, R = 1000, 16, 64, 530
    cu = np.concatenate([[0], np.cumsum(np.tile([2, 3], n // 2 * R))]).astype(np.int32)
    T = int(cu[-1]) // R
    qkv = torch.randn((T, 3 * H * dh), generator=torch.Generator().manual_seed(3)).to(torch.bfloat16).to(DEV)
    out = torch.zeros((R * T, H * dh), dtype=torch.bfloat16, device=DEV)
    exe.exe_op_prefill_attention(BF16, cu, qkv.repeat(R, 1), H, dh, 0.125, 1, None, 0, out, force_generic=-1)
    one = torch.zeros((T, H * dh), dtype=torch.bfloat16, device=DEV)
    exe.exe_op_prefill_attention(BF16, cu[:n + 1], qkv, H, dh, 0.125, 1, None, 0, one, force_generic=-1)
    torch.cuda.synchronize()
    assert bool((one != 0).any(dim=1).all()) and bool((out.reshape(R, T, -1) == one).all())
