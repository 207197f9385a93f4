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
