"""Greedy argmax: rows at the edges of what its workgroup takes at a time, and the longest rows an int32 length allows."""
import pytest
import torch

import paper_2404_07947_amd as exe

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 1024, 1025, 4092, 4095, 4096, 4100, 4097, 16384, 16385, 16388, 50272])
@pytest.mark.parametrize("rows", [1, 5])
def test_every_position_and_the_lowest_on_ties(n, rows):
    g = torch.Generator().manual_seed(n)
    x = torch.randn((rows, n), generator=g)
    best = torch.randint(0, n, (rows, 3), generator=g)
    for r in range(rows):
        x[r, best[r]] = 9.0                                # up to three equal maxima
    x[-1, n - 1] = 10.0
    out = torch.zeros((rows,), dtype=torch.int32, device=DEV)
    exe.exe_op_argmax(x.to(DEV), rows, n, out)
    want = [int(best[r].min()) for r in range(rows)]
    want[-1] = n - 1
    assert out.cpu().tolist() == want
    nan = torch.full((rows, n), float("nan"), device=DEV)
    exe.exe_op_argmax(nan, rows, n, out)
    assert out.cpu().tolist() == [0] * rows
    low = torch.full((rows, n), float("-inf"), device=DEV)
    exe.exe_op_argmax(low, rows, n, out)
    assert out.cpu().tolist() == [0] * rows


@pytest.mark.parametrize("n", [2 ** 31 - 1025, 2 ** 31 - 1024])
def test_rows_close_to_the_longest(n):
    """Indexes of the last steps pass 2^31: vector loads (n a multiple of 4) and single ones.  One row is 8.6 GB."""
    print("argmax row of", n, flush=True)
    x = torch.zeros((n,), device=DEV)
    x[n - 1] = 1.0
    x[n - 7] = 1.0
    out = torch.zeros((1,), dtype=torch.int32, device=DEV)
    exe.exe_op_argmax(x, 1, n, out)
    assert int(out.item()) == n - 7
