"""The norm fused into the product behind it (up to 16 rows): a batch's logits at the row counts around the fused kernel's
edges against the oracle, for LayerNorm and RMSNorm models, float and bf16, encode and decode."""
import numpy as np
import pytest
import torch

import workload as wl
from gpu_util import DEV, make_pair, row_relerr

pytestmark = pytest.mark.gpu
N_SEQ = [1, 3, 8, 9, 16, 17]


@pytest.mark.parametrize("n", N_SEQ)
@pytest.mark.parametrize("dtype", [wl.DTYPE_F32, wl.DTYPE_BF16])
def test_decoder_only(n, dtype):
    shape = wl.tiny_shape().replace(dtype=dtype)
    m, o, _ = make_pair(shape, 5)
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 3, size=n).astype(np.int32) if n <= 9 else np.ones(n, np.int32)   # few-row encode batches as well
    prompts = [rng.integers(0, shape.vocab, size=k).astype(np.int32) for k in lens]
    out = torch.zeros((n, shape.vocab), dtype=torch.float32, device=DEV)
    m.encode(np.arange(n), lens, np.concatenate(prompts), out_device=out)
    got, ref = [out.cpu().numpy()], [np.stack([o.encode(i, p)[1] for i, p in enumerate(prompts)])]
    for t in range(2):
        fed = rng.integers(0, shape.vocab, size=n).astype(np.int32)
        m.decode_step(np.arange(n), fed, lens + t + 1, out_device=out)
        got.append(out.cpu().numpy())
        ref.append(np.stack([o.decode(i, int(fed[i]))[1] for i in range(n)]))
    m.close()
    assert row_relerr(np.stack(got), np.stack(ref)) < (1e-4 if dtype == wl.DTYPE_F32 else 2e-2)


@pytest.mark.parametrize("n", N_SEQ)
@pytest.mark.parametrize("dtype", [wl.DTYPE_F32, wl.DTYPE_BF16])
def test_encoder_decoder(n, dtype):
    shape = wl.small_t5_shape(dtype)
    m, o, _ = make_pair(shape, 6)
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 12, size=n).astype(np.int32)
    prompts = [rng.integers(0, shape.vocab, size=k).astype(np.int32) for k in lens]
    m.encode(np.arange(n), lens, np.concatenate(prompts), reserve_lengths=np.full(n, 8, np.int32))
    for i, p in enumerate(prompts):
        o.encode(i, p)
    out = torch.zeros((n, shape.vocab), dtype=torch.float32, device=DEV)
    got, ref = [], []
    for t in range(3):
        fed = rng.integers(0, shape.vocab, size=n).astype(np.int32)
        m.decode_step(np.arange(n), fed, np.full(n, t + 1, np.int32), out_device=out)
        got.append(out.cpu().numpy())
        ref.append(np.stack([o.decode(i, int(fed[i]))[1] for i in range(n)]))
    m.close()
    assert row_relerr(np.stack(got), np.stack(ref)) < (1e-4 if dtype == wl.DTYPE_F32 else 2e-2)
