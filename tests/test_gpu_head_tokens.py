"""The tokens of a small model's calls against the logits they return: vocabularies at the edges of the LM head's 16 features a
workgroup, rows at the edges of its 8 and 16 a workgroup and of the limits beyond which a kernel of its own picks them, equal logits (the lowest index), rows of NaN and of infinities."""
import numpy as np
import pytest
import torch

import paper_2404_07947_amd as exe
import workload as wl
from gpu_util import DEV, kv_bytes_per_token

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8, 9, 16, 17, 33])
@pytest.mark.parametrize("vocab,dtype", [(16, wl.DTYPE_F32), (260, wl.DTYPE_BF16), (1028, wl.DTYPE_F32), (2048, wl.DTYPE_BF16), (4096, wl.DTYPE_F32)])
@pytest.mark.parametrize("kind", ["plain", "ties", "nan", "all_nan", "inf"])
def test_tokens_are_the_argmax_of_the_logits(n, vocab, dtype, kind):
    shape = wl.tiny_shape().replace(n_layers=1, vocab=vocab, max_pos=64, dtype=dtype)
    w = [t.to(DEV) for t in wl.make_weights(shape, 3)]
    emb = next(t for t in w if tuple(t.shape) == (vocab, shape.d_model))
    rng = np.random.default_rng(n)
    used = 4                                               # the tokens that are fed; the others' rows are free to change
    if kind == "ties":
        emb[used:] = emb[used:used + 3].repeat(-(-vocab // 3), 1)[:vocab - used] * 40
    elif kind == "nan":
        emb[torch.from_numpy(rng.permutation(np.arange(used, vocab))[:vocab // 2])] = float("nan")
    elif kind == "all_nan":
        emb[used:] = float("nan")
        emb[:used, 0] = float("nan")                       # and with them the rows themselves
    elif kind == "inf":
        emb[used:, 0] = torch.from_numpy(rng.choice([np.inf, -np.inf], size=vocab - used)).to(emb)
    cfg = exe.config_from_shape(shape, kv_pool_bytes=4096 * kv_bytes_per_token(shape), max_seqs=64, max_batch_tokens=512, max_batch_seqs=64)
    m = exe.Model(cfg, w)
    lens = rng.integers(1, 8, size=n).astype(np.int32)
    out = torch.zeros((n, vocab), dtype=torch.float32, device=DEV)
    print(f"head tokens n={n} vocab={vocab} {kind}", flush=True)

    def check(tokens):
        logits = out.cpu().numpy()
        low = np.where(np.isnan(logits), -np.inf, logits)
        want = np.where(np.isnan(logits).all(axis=1), 0, low.argmax(axis=1))
        for r in np.nonzero(np.isneginf(low.max(axis=1)) & ~np.isnan(logits).all(axis=1))[0]:
            want[r] = np.nonzero(~np.isnan(logits[r]))[0][0]
        assert np.array_equal(tokens, want)
        if kind == "ties":                                 # they are met: the largest logit is there more than once, or of a fed token
            assert n < 8 or max((logits == logits.max(axis=1, keepdims=True)).sum(axis=1)) > 1

    check(m.encode(np.arange(n), lens, rng.integers(0, used, size=int(lens.sum())).astype(np.int32), reserve_lengths=lens + 3, out_device=out))
    for t in range(2):
        check(m.decode_step(np.arange(n), rng.integers(0, used, size=n).astype(np.int32), lens + t + 1, out_device=out))
    m.close()


@pytest.mark.parametrize("vocab,n", [(2048, 4), (1028, 15), (2048, 12), (32000, 5)])
def test_outputs_are_complete_on_return(vocab, n):
    """When a call that returns tokens is back, its stream is idle, and another stream that reads the logits right behind it finds
    all of them (entries of the LM head's workgroups, and argmax_kernel)."""
    shape = wl.tiny_shape().replace(n_layers=1, vocab=vocab, max_pos=512)
    w = [t.to(DEV) for t in wl.make_weights(shape, 3)]
    cfg = exe.config_from_shape(shape, kv_pool_bytes=16384 * kv_bytes_per_token(shape), max_seqs=16, max_batch_tokens=256, max_batch_seqs=16)
    stream, other = torch.cuda.Stream(), torch.cuda.Stream()
    m = exe.Model(cfg, w, stream=stream)
    rng = np.random.default_rng(n)
    lens = rng.integers(1, 8, size=n).astype(np.int32)
    out = torch.empty((n, vocab), dtype=torch.float32, device=DEV)
    m.encode(np.arange(n), lens, rng.integers(0, vocab, size=int(lens.sum())).astype(np.int32), reserve_lengths=lens + 100)
    assert stream.query(), "busy behind encode"
    for t in range(100):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        tokens = m.decode_step(np.arange(n), rng.integers(0, vocab, size=n).astype(np.int32), lens + t + 1, out_device=out)
        idle = stream.query()
        with torch.cuda.stream(other):
            seen = out.clone().cpu()                       # on `other`, which the copy to the host waits for
        assert idle, t
        assert np.array_equal(tokens, seen.numpy().argmax(axis=1)), t
        torch.cuda.synchronize()
        assert torch.equal(seen, out.cpu()), t
    m.close()


def test_many_short_calls():
    """Calls right behind one another, with no other synchronisation between them: every call's tokens are the argmax of its own logits."""
    shape = wl.tiny_shape().replace(n_layers=1, vocab=2048, max_pos=512)
    w = [t.to(DEV) for t in wl.make_weights(shape, 3)]
    n, calls = 4, 400
    cfg = exe.config_from_shape(shape, kv_pool_bytes=16384 * kv_bytes_per_token(shape), max_seqs=16, max_batch_tokens=256, max_batch_seqs=16)
    m = exe.Model(cfg, w, stream=torch.cuda.Stream())
    rng = np.random.default_rng(n)
    lens = np.full(n, 5, dtype=np.int32)
    fed = rng.integers(0, shape.vocab, size=(calls, n)).astype(np.int32)
    out = torch.full((calls, n, shape.vocab), float("nan"), device=DEV)
    torch.cuda.synchronize()
    m.encode(np.arange(n), lens, rng.integers(0, shape.vocab, size=5 * n).astype(np.int32), reserve_lengths=lens + calls)
    tokens = [m.decode_step(np.arange(n), fed[t], lens + t + 1, out_device=out[t]) for t in range(calls)]
    assert np.array_equal(np.stack(tokens), out.cpu().numpy().argmax(axis=2))
    m.close()
