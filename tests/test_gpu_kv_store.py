"""Keys and values that an encode batch's projections store into the cache themselves: bit for bit those that the copy kernel
writes (a paged pool's encode runs it), for batches whose projection is one launch, two, or too small to do it."""
import numpy as np
import pytest
import torch

import paper_2404_07947_amd as exe
import workload as wl
from gpu_util import DEV, kv_bytes_per_token

pytestmark = pytest.mark.gpu


def shape_of(dtype, dh, layers=2):
    # 8 heads: 3 * 8 * dh features, 1536 and 3072: keys begin at the border of a tile of 256, values too
    return wl.tiny_shape().replace(n_layers=layers, d_model=512, n_heads=8, head_dim=dh, d_ff=512, vocab=512, max_pos=1024, dtype=dtype)


def model_of(shape, w, tokens, seqs, block=0):
    cfg = exe.config_from_shape(shape, kv_pool_bytes=(tokens + seqs * 300) * 2 * kv_bytes_per_token(shape), max_seqs=seqs,
                                max_batch_tokens=tokens, max_batch_seqs=seqs, kv_block_size=block)
    return exe.Model(cfg, w)


# rows: below what the tiles take, one past a tile, several rounds of tiles with a remainder; in bf16 cut into two launches of which
# the second, of a row, does not store (5377 rows of 3072 features, 10753 of 1536)
@pytest.mark.parametrize("lens", [[3, 40], [257], [700, 333, 1, 90], [1000] * 9 + [129, 64, 1], [1000] * 5 + [375, 2], [1000] * 10 + [750, 3]],
                         ids=["few", "one", "ragged", "many", "cut", "cut_narrow"])
@pytest.mark.parametrize("dtype,dh", [(wl.DTYPE_F32, 64), (wl.DTYPE_F32, 128), (wl.DTYPE_BF16, 64), (wl.DTYPE_BF16, 128)])
def test_cache_bits_and_logits(dtype, dh, lens):
    shape = shape_of(dtype, dh)
    w = [t.to(DEV) for t in wl.make_weights(shape, 5)]
    n, total = len(lens), sum(lens)
    toks = wl.random_tokens(np.random.default_rng(3), total, shape.vocab)
    got = []
    for block in (0, 16):
        m = model_of(shape, w, total, n, block)
        print(f"kv store dtype={dtype} dh={dh} lens={lens} block={block}", flush=True)
        logits = torch.zeros((n, shape.vocab), device=DEV)
        m.encode(np.arange(n), np.array(lens, dtype=np.int32), toks, out_device=logits)
        got.append(([m.seq_export(i)[0] for i in range(n)], logits.cpu().numpy()))
        m.close()
    for i in range(n):
        assert np.array_equal(got[0][0][i], got[1][0][i]), i
    assert np.array_equal(got[0][1], got[1][1])


@pytest.mark.parametrize("dtype", [wl.DTYPE_F32, wl.DTYPE_BF16])
@pytest.mark.parametrize("lens", [[20, 9], [1200, 77, 1, 300], [1200, 77, 1, 823]], ids=["few", "many", "float_tiles"])
def test_cross_keys_and_values(dtype, lens):
    """Cross-attention keys and values are the projection of the returned encoder output, rounded once."""
    shape = wl.small_t5_shape(dtype)
    specs = [s[0] for s in wl.weight_specs(shape)]
    w = [t.to(DEV) for t in wl.make_weights(shape, 5)]
    n, total = len(lens), sum(lens)
    m = model_of(shape, w, total, n)
    out = torch.zeros((total, shape.d_model), dtype=w[0].dtype, device=DEV)
    m.encode(np.arange(n), np.array(lens, dtype=np.int32), wl.random_tokens(np.random.default_rng(3), total, shape.vocab),
             reserve_lengths=np.full(n, 8), out_device=out, want_tokens=False)
    o, t0 = out.double().cpu(), 0
    for i, L in enumerate(lens):
        buf, st = m.seq_export(i)
        assert st == {"kv_len": 0, "cross_len": L}
        kv = torch.from_numpy(buf.copy()).view(w[0].dtype).view(shape.n_dec_layers, 2, shape.n_heads, L, shape.head_dim).double()
        for l in range(shape.n_dec_layers):
            ref = (o[t0:t0 + L] @ w[specs.index(f"d{l}.w_xkv")].double().cpu().T).view(L, 2, shape.n_heads, shape.head_dim).permute(1, 2, 0, 3)
            # sums of 256 products in float: 256 * 2^-24 of the largest at most; bf16: half a unit of 8 bits on top
            tol = 2.0 ** -16 + (2.0 ** -8 if dtype == wl.DTYPE_BF16 else 0.0)
            assert float((kv[l] - ref).abs().max() / ref.abs().max()) < tol, (i, l)
        t0 += L


# rows and heads of 128 at which the QKV product is three launches and the second, of 256 rows, does not store (asserted in
# test_gemm_plans.py): counts at the GPT-3-175B width, and a long batch of a narrower one
@pytest.mark.parametrize("rows,heads", [(2049, 96), (2298, 96), (16385, 46)])
def test_a_launch_cut_twice(rows, heads):
    d = heads * 128
    shape = wl.gpt3_175b_share_shape(1).replace(d_model=d, n_heads=heads, d_ff=512)
    print(f"kv store rows={rows} heads={heads}", flush=True)
    w = wl.make_weights(shape, 5, device=DEV)
    lens = np.array([700, 333, 1, rows - 1034], dtype=np.int32)
    x = torch.randn((rows, d), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV).bfloat16()
    got = []
    for block in (0, 16):
        m = model_of(shape, w, rows, 4, block)
        out = torch.zeros((rows, d), dtype=torch.bfloat16, device=DEV)
        m.encode(np.arange(4), lens, None, hidden_in=x, want_tokens=False, out_device=out)
        got.append(([m.seq_export(i)[0] for i in range(4)], out.cpu()))
        m.close()
    for i in range(4):
        assert np.array_equal(got[0][0][i], got[1][0][i]), i
    assert torch.equal(got[0][1], got[1][1])


# 512 rows in one launch that stores.  Tiles of 256 x 160 (configuration 8): waves of 80 features, one of which holds the last queries
# and the first keys (20352 = 3 x 6784, 6784 = 84.8 x 80); of 256 x 128 (5): waves of 64, keys begin inside a tile.  The last tile is not full.
@pytest.mark.parametrize("dh,heads,cfg", [(128, 53, 8), (64, 106, 8), (64, 81, 5)])
def test_tiles_whose_waves_straddle_heads(dh, heads, cfg):
    """A paged pool's entries are copied out of the output."""
    rows, d = 512, heads * dh
    assert exe.exe_op_gemm_model_plan(wl.DTYPE_BF16, rows, 3 * d, d) == [{"rows": rows, "route": 0, "cfg": cfg, "splits": 1, "large": 1}]
    assert exe.exe_op_gemm_kv_plan(wl.DTYPE_BF16, rows, 3 * d, d) == ([(rows, 1)], rows)
    shape = wl.gpt3_175b_share_shape(1).replace(d_model=d, n_heads=heads, head_dim=dh, d_ff=512)
    w = wl.make_weights(shape, 5, device=DEV)
    lens = np.array([200, 133, 1, 178], dtype=np.int32)
    x = torch.randn((rows, d), generator=torch.Generator(device=DEV).manual_seed(3), device=DEV).bfloat16()
    got = []
    for block in (0, 16):
        m = model_of(shape, w, rows, 4, block)
        out = torch.zeros((rows, d), dtype=torch.bfloat16, device=DEV)
        m.encode(np.arange(4), lens, None, hidden_in=x, want_tokens=False, out_device=out)
        got.append([m.seq_export(i)[0] for i in range(4)] + [out.cpu().view(torch.int16).numpy()])
        m.close()
    assert all(np.array_equal(a, b) for a, b in zip(*got))
