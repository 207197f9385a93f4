"""Launch plans of the GEMMs (host logic: no GPU)."""
import threading

import pytest

import paper_2404_07947_amd as exe
import workload as wl

F32, BF16 = wl.DTYPE_F32, wl.DTYPE_BF16


def in_a_new_thread(fn):
    """Plans are remembered per thread: what a thread that has planned nothing yet gives."""
    out = []
    t = threading.Thread(target=lambda: out.append(fn()))
    t.start()
    t.join()
    return out[0]


@pytest.mark.parametrize("dtype", [BF16, F32])
@pytest.mark.parametrize("first,second", [((16, 1024, 1024), (16 + (1 << 18), 1024, 1024)),
                                          ((16, 1024, 1024), (16 + (1 << 20), 1024, 1024)),
                                          ((300, 1028, 64), (300, 1024, 64 + (1 << 23))),
                                          ((9, 512, 512), (8, 512 + (1 << 22), 512))])
def test_a_plan_does_not_depend_on_the_shapes_planned_before(dtype, first, second):
    def ask(shape):
        return exe.exe_op_gemm_plan(dtype, *shape), exe.exe_op_gemm_workspace(dtype, *shape)
    for a, b in ((first, second), (second, first)):
        assert in_a_new_thread(lambda: (ask(a), ask(b))[1]) == in_a_new_thread(lambda: ask(b))
