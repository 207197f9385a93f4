"""Decode attention's launch shapes: 4, 8 or 16 waves per row by the batch's lengths, and one workgroup per CU for long ragged ones.
For every type and head size, extent and paged, mean lengths that pick each shape in turn: a sequence's logits are compared with
the oracle and may not depend on the batch-mates whose lengths pick the shape."""
import numpy as np
import pytest
import torch

import workload as wl
from gpu_util import DEV, make_pair, row_relerr

pytestmark = pytest.mark.gpu
F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16


@pytest.mark.parametrize("block", [0, 16])
@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("dh", [64, 128])
def test_logits_do_not_depend_on_the_launch_shape(dtype, dh, block):
    size = 4 if dtype == F32 else 2
    step = 2 * 1024 // (dh * size)                       # rows a wave takes at a time: two loads of 1 KB
    # (few workgroups) up to 4 steps: 4 waves, up to 16: 8, else 16; from 256 KB of keys and values a row on one workgroup per CU
    means = [2 * step, 8 * step, 24 * step, (256 << 10) // (2 * dh * size) * 11 // 10]
    assert 24 * step * 2 * dh * size < 256 << 10
    shape = wl.tiny_shape().replace(max_pos=2048, n_heads=256 // dh, head_dim=dh, dtype=dtype)
    own, steps, mates = np.array([1, 3, 40]), 3, 9                                       # the sequences compared
    rng = np.random.default_rng(3)
    prompts = [rng.integers(0, shape.vocab, size=n).astype(np.int32) for n in own]
    fed = rng.integers(0, shape.vocab, size=(steps, len(own))).astype(np.int32)
    runs, ref = [], None
    for mean in means:
        mate = max(1, round(((mean - 2) * (len(own) + mates) - int(own.sum())) / mates))
        m, o, _ = make_pair(shape, 11, pool_tokens=mates * (mate + 40) + 256, kv_block_size=block)
        lens = np.concatenate([own, [mate] * mates])
        assert abs(lens.mean() + 2 - mean) <= 2 or mate == 1
        tokens = np.concatenate(prompts + [np.zeros(mates * mate, np.int32)])
        ids = np.arange(len(lens))
        for b in range(0, len(lens), 2):
            off = int(lens[:b].sum())
            m.encode(ids[b:b + 2], lens[b:b + 2], tokens[off:off + int(lens[b:b + 2].sum())], reserve_lengths=lens[b:b + 2] + 4)
        out = torch.zeros((len(lens), shape.vocab), dtype=torch.float32, device=DEV)
        parts = []
        for t in range(steps):
            m.decode_step(ids, np.concatenate([fed[t], np.zeros(mates, np.int32)]), lens + t + 1, out_device=out)
            parts.append(out[:len(own)].cpu().numpy())
        m.close()
        runs.append(np.stack(parts))
        if ref is None:
            for i, p in enumerate(prompts):
                o.encode(i, p)
            ref = np.stack([np.stack([o.decode(i, int(fed[t, i]))[1] for i in range(len(own))]) for t in range(steps)])
    # float: sums in another order; bf16: roundings between the layers may fall the other way
    tol = 1e-5 if dtype == F32 else 2e-2
    for mean, got in zip(means, runs):
        assert row_relerr(got, ref) < (1e-4 if dtype == F32 else 2e-2), mean
        assert np.max(np.abs(got - runs[0])) < tol * np.max(np.abs(runs[0])), mean
