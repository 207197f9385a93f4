"""exe_kernel_times: the bytes that the launches of a class book."""
import numpy as np
import pytest

import paper_2404_07947_amd as exe
import workload as wl
from gpu_util import DEV, make_pair

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 8, 150])
@pytest.mark.parametrize("hidden", [0, 1])
def test_residual_traffic_is_booked_by_the_launch_that_moves_it(n, hidden):
    """A projection into the residual stream may leave split-K partial sums for the norm behind it.  Per such pair the products
    book splits * 4 bytes an element in place of the 8 of a read and a write, the norm splits * 4 more and the write of the
    finished row: 12 bytes an element between them, whatever the splits.  Hidden states out: a reduction finishes the last row."""
    import torch
    d, f, L = 1024, 16384, 2
    shape = wl.tiny_shape().replace(n_layers=L, d_model=d, n_heads=8, head_dim=128, d_ff=f, max_pos=64, dtype=wl.DTYPE_BF16)
    if hidden:
        shape = shape.replace(has_embed=0, has_lm_head=0, vocab=0, pos=wl.POS_NONE, max_pos=0)
    m, _, _ = make_pair(shape, 5, pool_tokens=16 * 160, max_seqs=160, max_batch_seqs=160)
    ids, lens = np.arange(n), np.full(n, 3)
    toks = None if hidden else np.zeros(3 * n, np.int32)
    x = torch.zeros((3 * n, d), dtype=torch.bfloat16, device=DEV) if hidden else None
    m.encode(ids, lens, toks, reserve_lengths=lens + 4, hidden_in=x, want_tokens=not hidden)
    m.kernel_timing(True)
    out = torch.zeros((n, d), dtype=torch.bfloat16, device=DEV) if hidden else None
    m.decode_step(ids, None if hidden else np.zeros(n, np.int32), lens + 1, hidden_in=x[:n] if hidden else None,
                  want_tokens=not hidden, out_device=out)
    k = {r["kind"]: r for r in m.kernel_times()}
    m.close()
    inner, V = 1024, 0 if hidden else shape.vocab
    gemm = L * 2 * ((n * d + 3 * inner * d + n * 3 * inner) + (n * inner + d * inner) + (n * d + f * d + n * f) + (n * f + d * f))
    gemm += L * 2 * 8 * n * d + (2 * (n * d + V * d) + 4 * n * V)
    extra_gemm = k["gemm_skinny"]["bytes"] - (gemm - (2 * n * d if hidden else 0))
    extra_norm = k["norm"]["bytes"] - (2 * L + (0 if hidden else 1)) * n * d * 6
    if hidden:                                            # the reduction reads and writes the row itself, the norm reads it anyway
        moved = k["other"]["bytes"] - 2 * n * d * 6
        assert moved >= 0
        extra_norm += moved - (4 * n * d if moved else 0)
    pairs = (extra_norm - extra_gemm) / (12 * n * d)
    assert pairs == round(pairs) and 1 <= pairs <= 2 * L, (pairs, extra_gemm, extra_norm)
