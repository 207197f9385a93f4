"""Prefill attention on inputs that separate the MFMA kernel from plain arithmetic: what a row may not depend on, and what its
probabilities have to keep."""
import numpy as np
import pytest
import torch

import paper_2404_07947_amd as exe
import workload as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16
TYPES = [(BF16, 64), (BF16, 128), (F32, 64), (F32, 128)]


def td(dtype):
    return torch.float32 if dtype == F32 else torch.bfloat16


def run(dtype, dh, H, lens, qkv, scale, causal, tab=None, R=0, generic=-1):            # -1: the MFMA kernel, whatever the size
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    out = torch.zeros((int(cu[-1]), H * dh), dtype=td(dtype), device=DEV)
    exe.exe_op_prefill_attention(dtype, cu, qkv.to(DEV), H, dh, scale, causal, None if tab is None else tab.to(DEV), R, out,
                                 force_generic=generic)
    torch.cuda.synchronize()
    return out.float().cpu().numpy()


def reference(dh, H, lens, qkv, scale, causal, tab=None, R=0):
    """Row by row in 64 bits, from the keys and values that a row attends to and no others."""
    x, inner, t0, rows = qkv.double().numpy(), H * dh, 0, []
    for L in lens:
        s = x[t0:t0 + L]
        for i in range(L):
            n, row = (i + 1 if causal else L), []
            for h in range(H):
                q, k, v = (s[:, j * inner + h * dh:j * inner + (h + 1) * dh] for j in range(3))
                sc = (k[:n] @ q[i]) * float(np.float32(scale))
                if tab is not None:
                    sc = sc + tab.double().numpy()[h][np.clip(np.arange(n) - i, -R, R) + R]
                p = np.exp(sc - sc.max())
                with np.errstate(invalid="ignore"):
                    row.append((p / p.sum()) @ v[:n])
            rows.append(np.concatenate(row))
        t0 += L
    return np.stack(rows)


def tolerance(dtype):
    return 1e-5 if dtype == F32 else 2.0 ** -7          # as in test_gpu_prefill_types.py; bf16 x 128 rounds the probabilities too


@pytest.mark.parametrize("dtype,dh", TYPES)
@pytest.mark.parametrize("use_bias", [0, 1])
def test_causal_rows_do_not_see_later_values(dtype, dh, use_bias):
    """Infinite and NaN value rows late in a sequence (and in its neighbour): every earlier row stays finite and right, the
    rows from there on have them in the features that hold them and nowhere else."""
    H, lens, R = 2, [200, 70], 40
    g = torch.Generator().manual_seed(dh)
    qkv = torch.randn((270, 3 * H * dh), generator=g).to(td(dtype))
    tab = torch.randn((H, 2 * R + 1), generator=g) * 0.5 if use_bias else None
    ref = reference(dh, H, lens, qkv, 0.1, 1, tab, R)
    bad = qkv.clone()
    bad[130, 2 * H * dh:] = float("inf")                # all features: row 130 is in the key tile of rows 128 .. 191
    bad[199, 2 * H * dh + 3] = float("nan")             # the last row of the sequence
    bad[200 + 33, 2 * H * dh + dh + 5] = float("-inf")  # one feature of head 1
    got = run(dtype, dh, H, lens, bad, 0.1, 1, tab, R)
    clean = np.ones(270, bool)
    clean[130:200] = clean[233:] = False
    err = np.abs(got[clean] - ref[clean]).max(axis=1) / np.abs(ref[clean]).max(axis=1)
    assert err.max() < tolerance(dtype), (int(err.argmax()), float(err.max()))
    assert np.all(np.isposinf(got[131:199])), "rows 131 .. 198 see the infinite row"
    other = np.ones(H * dh, bool)
    other[dh + 5] = False
    err = np.abs(got[233:, other] - ref[233:, other]).max(axis=1) / np.abs(ref[233:]).max(axis=1)
    assert err.max() < tolerance(dtype) and np.all(np.isneginf(got[234:, dh + 5]))


@pytest.mark.parametrize("dtype,dh", TYPES)
@pytest.mark.parametrize("scale", [-3.0, 0.0])
@pytest.mark.parametrize("causal,use_bias", [(1, 0), (0, 1)])
def test_scales_that_are_not_positive(dtype, dh, scale, causal, use_bias):
    H, lens, R = 2, [200, 17], 40
    g = torch.Generator().manual_seed(7 + dh)
    qkv = torch.randn((217, 3 * H * dh), generator=g).to(td(dtype))
    tab = torch.randn((H, 2 * R + 1), generator=g) * 0.5 if use_bias else None
    ref = reference(dh, H, lens, qkv, scale, causal, tab, R)
    got = run(dtype, dh, H, lens, qkv, scale, causal, tab, R)
    err = np.abs(got - ref).max(axis=1) / np.abs(ref).max(axis=1)
    # a score is 3 times a float sum of dh products of up to about 10, |.| 150 at most in all: 3 * 150 * 2^-24 relative in p
    assert err.max() < (5e-5 if dtype == F32 else 2.0 ** -7), (int(err.argmax()), float(err.max()))


@pytest.mark.parametrize("dtype,dh", [(BF16, 64), (F32, 64), (F32, 128)])
@pytest.mark.parametrize("generic", [-1, 1])
def test_probabilities_keep_24_bits(dtype, dh, generic):
    """Two keys whose values nearly cancel: a feature's result is p0 * a - p1 * b with |result| down to 2^-16 of its terms, so
    a probability rounded to fewer bits shows however the result itself is stored."""
    n = 400                                              # sequences of two rows; the second row of each is compared
    g = torch.Generator().manual_seed(3)
    qkv = torch.zeros((2 * n, 3 * dh))
    qkv[:, :2 * dh] = (torch.randn((2 * n, 2 * dh), generator=g) * 0.3).to(torch.bfloat16).float()
    x = qkv.double().numpy().reshape(n, 2, 3 * dh)
    s = np.einsum("nd,nkd->nk", x[:, 1, :dh], x[:, :, dh:2 * dh]) * 0.125
    ratio = np.exp(s[:, 0] - s[:, 1])                    # p0 / p1
    a = np.arange(128, 256) / 128.0                      # every bf16 value in [1, 2), and in [0.25, 4) for b
    b = np.concatenate([a / 4, a / 2, a, a * 2])
    V = np.zeros((n, 2, dh))
    for i in range(n):
        off = np.abs(ratio[i] * a[:, None] - b[None, :])
        best = np.argsort(off, axis=None)[:dh]
        V[i, 0], V[i, 1] = a[best // len(b)], -b[best % len(b)]
    qkv = qkv.view(n, 2, 3 * dh)
    qkv[:, :, 2 * dh:] = torch.from_numpy(V).float()
    qkv = qkv.reshape(2 * n, 3 * dh).to(td(dtype))
    lens = [2] * n
    got, ref = run(dtype, dh, 1, lens, qkv, 0.125, 1, generic=generic)[1::2], reference(dh, 1, lens, qkv, 0.125, 1)[1::2]
    p1 = 1.0 / (1.0 + ratio)
    terms = (p1 * ratio)[:, None] * V[:, 0] - p1[:, None] * V[:, 1]                  # |p0 a| + |p1 b|
    assert np.mean(np.abs(ref) / terms < 2.0 ** -11) > 0.25          # where the rounding of a bf16 result hides no 2^-18
    # a float exponential and float sums are good to a few 2^-24 of the terms (2^-21 taken); 16-bit probabilities to 2^-18
    bound = 2.0 ** -21 * terms + (0 if dtype == F32 else 2.0 ** -8) * np.abs(ref)
    assert np.all(np.abs(got - ref) < bound), float(np.max(np.abs(got - ref) / terms))


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("n,causal,R", [(300, 1, 0), (1000, 1, 0), (1000, 0, 127)])
def test_float_sums_are_as_good_as_the_row_kernels(dh, n, causal, R):
    """Against 64 bits: the MFMA kernel's sums may err no more than those of the row kernel, which adds up short chains in a
    tree (with one chain per score and one per output it erred 2.3 to 3.3 times as much)."""
    H = 4
    g = torch.Generator().manual_seed(n + dh)
    qkv = torch.randn((n, 3 * H * dh), generator=g) * 1.5
    tab = torch.randn((H, 2 * R + 1), generator=g) if R else None
    scale = float(np.float32(1.0 / np.sqrt(dh)))
    x, ref = qkv.double().numpy(), np.zeros((n, H * dh))
    i, j = np.arange(n)[:, None], np.arange(n)[None, :]
    for h in range(H):
        q, k, v = (x[:, c * H * dh + h * dh:c * H * dh + (h + 1) * dh] for c in range(3))
        s = q @ k.T * scale
        if R:
            s += tab.double().numpy()[h][np.clip(j - i, -R, R) + R]
        if causal:
            s = np.where(j <= i, s, -np.inf)
        p = np.exp(s - s.max(axis=1, keepdims=True))
        ref[:, h * dh:(h + 1) * dh] = (p / p.sum(axis=1, keepdims=True)) @ v
    err = [np.linalg.norm(run(F32, dh, H, [n], qkv, scale, causal, tab, R, generic) - ref) / np.linalg.norm(ref) for generic in (-1, 1)]
    # measured 0.93 to 1.06; two errors of the same make over 77 000 and more outputs differ by far less than a quarter
    assert err[0] < 1.25 * err[1], err
