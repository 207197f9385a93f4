"""Decode iterations of small models (a launch per attention and feed-forward block) against the oracle: the edges of its row
counts, widths, head sizes and slices, float and bf16, LayerNorm and RMSNorm, with and without embedding, one to three layers."""
import numpy as np
import pytest
import torch

import workload as wl
from gpu_util import DEV, make_pair, row_relerr, tdtype

pytestmark = pytest.mark.gpu
F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16
# per-row bounds of the model tests: float sums of up to 2048 terms, bf16 roundings of a few layers
TOL = {F32: 1e-4, BF16: 2e-2}


def decoder_only(dtype, d, H, dh, f, layers, hidden):
    s = wl.tiny_shape().replace(n_layers=layers, d_model=d, n_heads=H, head_dim=dh, d_ff=f, vocab=260, max_pos=512, dtype=dtype)
    return s.replace(has_embed=0, has_lm_head=0, vocab=0, pos=wl.POS_NONE, max_pos=0) if hidden else s


# (rows at and beyond the blocks' 16 and the limit of 32), widths from one chunk of 256 bytes to four, one slice of 64 to 32.  Beyond
# 12 rows the two last shapes in bf16, 512 wide with 512 features of all heads, run as launches of their own: see the work limit below.
@pytest.mark.parametrize("n", [1, 2, 16, 17, 32, 33])
@pytest.mark.parametrize("dtype,d,H,dh,f,layers,hidden", [
    (F32, 64, 1, 64, 64, 1, 0), (F32, 192, 3, 64, 2048, 2, 0), (F32, 256, 2, 128, 320, 3, 0), (F32, 256, 4, 64, 1024, 2, 1),
    (BF16, 128, 2, 64, 128, 1, 0), (BF16, 384, 5, 64, 576, 2, 0), (BF16, 512, 4, 128, 2048, 3, 0), (BF16, 512, 8, 64, 1024, 2, 1)])
def test_decoder_only(n, dtype, d, H, dh, f, layers, hidden):
    shape = decoder_only(dtype, d, H, dh, f, layers, hidden)
    print(f"small decode n={n} {shape}", flush=True)
    m, o, _ = make_pair(shape, 5, pool_tokens=8192)
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 12, size=n).astype(np.int32)
    lens[0] = 1
    lens[-1] = 300                                # more cached rows than a pass of the 16 waves takes
    steps, T = 3, int(lens.sum())
    td = tdtype(shape)
    toks = None if hidden else rng.integers(0, shape.vocab, size=T).astype(np.int32)
    x = torch.randn((T + steps * n, d), generator=torch.Generator().manual_seed(n)).to(td) if hidden else None
    width = d if hidden else shape.vocab
    out = torch.zeros((n, width), dtype=td if hidden else torch.float32, device=DEV)
    m.encode(np.arange(n), lens, toks, reserve_lengths=lens + steps, hidden_in=x[:T].to(DEV) if hidden else None, want_tokens=not hidden)
    t0 = 0
    for i, k in enumerate(lens):
        o.encode(i, None if hidden else toks[t0:t0 + k], x[t0:t0 + k].float().numpy() if hidden else None)
        t0 += k
    got, ref = [], []
    for t in range(steps):
        fed = None if hidden else rng.integers(0, shape.vocab, size=n).astype(np.int32)
        xt = x[T + t * n:T + (t + 1) * n] if hidden else None
        m.decode_step(np.arange(n), fed, lens + t + 1, hidden_in=xt.to(DEV) if hidden else None, want_tokens=not hidden, out_device=out)
        got.append(out.float().cpu().numpy())
        ref.append(np.stack([o.decode(i, 0 if hidden else int(fed[i]), xt[i].float().numpy() if hidden else None)[1] for i in range(n)]))
    m.close()
    assert row_relerr(np.stack(got), np.stack(ref)) < TOL[dtype]


@pytest.mark.parametrize("n", [1, 12, 16, 17, 32, 33])
@pytest.mark.parametrize("dtype,d,H,dh,f,layers,cross_bias", [(F32, 256, 4, 64, 512, 1, 1), (F32, 128, 2, 128, 64, 3, 0),
                                                              (BF16, 512, 3, 128, 1024, 1, 1), (BF16, 256, 4, 64, 512, 2, 1)])
def test_encoder_decoder(n, dtype, d, H, dh, f, layers, cross_bias):
    shape = wl.small_t5_shape(dtype).replace(n_layers=1, n_dec_layers=layers, d_model=d, n_heads=H, head_dim=dh, d_ff=f, vocab=260,
                                             cross_rel_bias=cross_bias)
    print(f"small decode n={n} {shape}", flush=True)
    m, o, _ = make_pair(shape, 6, pool_tokens=8192)
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 12, size=n).astype(np.int32)
    lens[-1] = 200
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
    assert row_relerr(np.stack(got), np.stack(ref)) < TOL[dtype]


# the limit of rows x heads x head size x width, 3 * 2^20, at 12 rows of 512 x 512 (and in float of 256 x 1024), and wide bf16 rows
# below it at more than 16 rows
EDGES = [(n, *k) for n in (12, 13) for k in ((BF16, 512, 4, 128), (BF16, 512, 8, 64), (F32, 256, 16, 64))]
EDGES += [(n, BF16, 512, H, 64) for n in (17, 32) for H in (1, 2, 3)] + [(17, BF16, 512, 5, 64), (18, BF16, 512, 5, 64), (19, BF16, 512, 5, 64), (20, BF16, 512, 5, 64), (17, BF16, 512, 2, 128)]


@pytest.mark.parametrize("n,dtype,d,H,dh", EDGES)
def test_at_the_work_limit(n, dtype, d, H, dh):
    test_decoder_only(n, dtype, d, H, dh, 1024, 2, 0)


@pytest.mark.parametrize("n,dtype,d,H,dh", EDGES + [(n, F32, 256, 4, 64) for n in (1, 32, 33)])
def test_which_launches_an_iteration_makes(n, dtype, d, H, dh):
    """A launch for the attention block and one for the feed-forward of each layer within the limits, else four products a layer."""
    layers = 2
    m, _, _ = make_pair(decoder_only(dtype, d, H, dh, 1024, layers, 0), 5, pool_tokens=8192)
    m.encode(np.arange(n), np.full(n, 3), np.zeros(3 * n, np.int32), reserve_lengths=np.full(n, 8))
    m.kernel_timing(True)
    m.decode_step(np.arange(n), np.zeros(n, np.int32), np.full(n, 4))
    k = {r["kind"]: r["launches"] for r in m.kernel_times()}
    m.close()
    fused = n <= 32 and n * H * dh * d <= 3 << 20
    assert k["decode_attn"] == layers and k["gemm_skinny"] == (1 if fused else 4) * layers + 1
