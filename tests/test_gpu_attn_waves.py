"""Decode attention's launch shapes (4, 8 or 16 waves per row, one or two workgroups per CU) against each other: a sequence's
logits may not depend on the batch-mates whose lengths pick the shape.  The 16-wave kernel is compared with the oracle in
test_gpu_ops.py; the model tests compare short batches with it as well."""
import numpy as np
import pytest
import torch

import workload as wl
from gpu_util import DEV, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("block", [0, 16])
@pytest.mark.parametrize("heads,dtype", [(4, wl.DTYPE_F32), (2, wl.DTYPE_F32), (4, wl.DTYPE_BF16), (2, wl.DTYPE_BF16)])
def test_logits_do_not_depend_on_the_launch_shape(heads, dtype, block):
    shape = wl.tiny_shape().replace(max_pos=1024, n_heads=heads, dtype=dtype)            # head size 64 or 128
    own = np.array([1, 3, 40])                                                           # the sequences compared
    rng = np.random.default_rng(3)
    prompts = [rng.integers(0, shape.vocab, size=n).astype(np.int32) for n in own]
    fed = rng.integers(0, shape.vocab, size=(3, len(own))).astype(np.int32)
    ref = None
    for mate in (1, 60, 180, 260, 1000):                                                 # mean lengths from 12 to 760
        m, _, _ = make_pair(shape, 11, pool_tokens=16384, kv_block_size=block)
        lens = np.concatenate([own, [mate] * 9])
        tokens = np.concatenate(prompts + [np.zeros(9 * mate, np.int32)])
        ids = np.arange(len(lens))
        parts = []
        for b in range(0, len(lens), 4):
            off = int(lens[:b].sum())
            m.encode(ids[b:b + 4], lens[b:b + 4], tokens[off:off + int(lens[b:b + 4].sum())], reserve_lengths=lens[b:b + 4] + 4)
        out = torch.zeros((len(lens), shape.vocab), dtype=torch.float32, device=DEV)
        for t in range(3):
            m.decode_step(ids, np.concatenate([fed[t], np.zeros(9, np.int32)]), lens + t + 1, out_device=out)
            parts.append(out[:len(own)].cpu().numpy())
        m.close()
        got = np.stack(parts)
        if ref is None:
            ref = got
        # float: sums in another order; bf16: one rounding of the attention output may fall the other way, and the batch size
        # (12 rows in every run) keeps the products' launches the same
        tol = 1e-5 if dtype == wl.DTYPE_F32 else 2e-2
        assert np.max(np.abs(got - ref)) < tol * np.max(np.abs(ref)), mate
