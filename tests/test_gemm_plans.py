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


@pytest.mark.parametrize("M", [1, 7, 128, 1000, 5000])
@pytest.mark.parametrize("N", [4, 128, 1024])
def test_float_rows_beyond_32_bit_offsets_take_the_kernel_with_64_bit_ones(M, N):
    """The MFMA kernels address a tile's rows by 32-bit byte offsets: 128 rows of 2^23 floats are 4 GB."""
    assert exe.exe_op_gemm_plan(F32, M, N, (1 << 23) - 32)["route"] != 2
    for K in (1 << 23, (1 << 23) + 32, 1 << 26):
        assert exe.exe_op_gemm_plan(F32, M, N, K)["route"] == 2


@pytest.mark.parametrize("dtype,K", [(F32, 1 << 24), (BF16, 1 << 25)])
def test_the_streaming_gemm_refuses_80_such_rows(dtype, K):
    assert exe.lib().exe_op_gemm_stream(None, dtype, 8, 128, K, 64, 64, None, -1, 1.0, 2, 64, 5, 1, 1, None, 0) == -2


# (features, depth) of the projections whose last features are keys and values: OPT-13B, the GPT-3-175B width, T5-11B's encoder and its
# cross keys and values, 1024 wide, 256 wide, and widths between
KV_SHAPES = [(15360, 5120), (36864, 12288), (49152, 1024), (32768, 1024), (3072, 1024), (768, 256)] + [(3 * d, d) for d in (5888, 8960, 11776, 13824)]


@pytest.mark.parametrize("N,K", KV_SHAPES)
@pytest.mark.parametrize("dtype", [BF16, F32])
def test_rows_counted_on_are_the_rows_stored(dtype, N, K):
    """A product of many rows is cut into launches, each part again where that pays; an encode call copies the keys and values behind
    those that it counts on.  Every token count to 20 000: the leading rows whose launches store are what it counts on, and a launch
    is not cut once more when it is made."""
    for M in range(1, 20001 if dtype == BF16 else 3001):
        launches, counted = exe.exe_op_gemm_kv_plan(dtype, M, N, K)
        assert sum(r for r, _ in launches) == M
        lead = next((i for i, (_, stores) in enumerate(launches) if not stores), len(launches))
        assert counted == sum(r for r, _ in launches[:lead]), (M, launches)
        for r, stores in launches if len(launches) > 1 else ():
            assert exe.exe_op_gemm_kv_plan(dtype, r, N, K)[0] == [(r, stores)], (M, launches)


def test_launches_that_the_cache_tests_run():
    """The counts that test_gpu_kv_store.py runs: in the middle of three launches 256 rows that do not store; two launches, the second
    of a row; float launches that store, from 2049 rows on."""
    assert exe.exe_op_gemm_kv_plan(BF16, 5377, 3072, 512) == ([(5376, 1), (1, 0)], 5376)
    assert exe.exe_op_gemm_kv_plan(BF16, 10753, 1536, 512) == ([(10752, 1), (1, 0)], 10752)
    assert exe.exe_op_gemm_kv_plan(F32, 2101, 512, 256) == ([(2101, 1)], 2101)
    assert exe.exe_op_gemm_kv_plan(BF16, 2049, 36864, 12288) == ([(1792, 1), (256, 0), (1, 0)], 1792)
    assert exe.exe_op_gemm_kv_plan(BF16, 2298, 36864, 12288) == ([(1792, 1), (256, 0), (250, 0)], 1792)
    assert exe.exe_op_gemm_kv_plan(BF16, 16385, 17664, 5888) == ([(16128, 1), (256, 0), (1, 0)], 16128)


@pytest.mark.parametrize("dtype", [BF16, F32])
def test_model_plans_are_the_launches(dtype):
    """The rows of exe_op_gemm_model_plan are those of the launches that are made, and forced plans are what was asked for."""
    for M, N, K in [(1, 1024, 1024), (300, 3072, 1024), (2049, 36864, 12288), (5377, 3072, 512), (16385, 17664, 5888)]:
        plans = exe.exe_op_gemm_model_plan(dtype, M, N, K)
        assert [p["rows"] for p in plans] == [r for r, _ in exe.exe_op_gemm_kv_plan(dtype, M, N, K)[0]]
        assert [p["route"] == 0 and p["splits"] == 1 and (dtype == F32 or p["large"] == 1) for p in plans] == \
            [bool(s) for _, s in exe.exe_op_gemm_kv_plan(dtype, M, N, K)[0]]
    assert exe.exe_op_gemm_model_plan(BF16, 300, 1024, 1024, 8, 2) == [{"rows": 300, "route": 0, "cfg": 8, "splits": 2, "large": 1}]
    assert exe.exe_op_gemm_model_plan(BF16, 300, 1024, 192, 5, 1) == [{"rows": 300, "route": 0, "cfg": 5, "splits": 1, "large": 0}]
    for bad in ((BF16, 300, 1024, 1024, 7, 1), (BF16, 300, 1024, 192, 8, 1), (F32, 300, 1024, 1024, 2, 1)):
        with pytest.raises(exe.ExeError):
            exe.exe_op_gemm_model_plan(*bad)


# us measured, gemm_tile_kernel / gemm_large_kernel: see runs_large in csrc/kernels_gemm.hip
@pytest.mark.parametrize("M,N,K,splits,large", [(256, 24576, 3072, 1, 1), (256, 24576, 6144, 1, 0), (512, 16384, 6144, 1, 1), (512, 16384, 12288, 1, 0),      # 51/51 99/107 94/94 188/218
                                                (768, 9216, 11008, 1, 1), (1024, 16384, 12288, 1, 1), (1024, 16384, 14336, 1, 0), (448, 15360, 11008, 1, 0),    # 153/150 342/324 402/439 158/173
                                                (224, 24576, 8192, 1, 0), (256, 9216, 4096, 3, 1), (256, 8192, 8192, 4, 0), (512, 5120, 12288, 3, 1),          # 122/141 36.7/35.5 48/51 75/73
                                                (512, 13824, 14336, 2, 0), (256, 10240, 20480, 3, 0), (1100, 5120, 20480, 1, 1), (300, 1024, 192, 1, 0)])       # 217/231 124/133
def test_tiles_of_256_x_128_run_on_the_faster_kernel(M, N, K, splits, large):
    assert exe.exe_op_gemm_model_plan(BF16, M, N, K, 5, splits)[0]["large"] == large
    assert exe.exe_op_gemm_model_plan(BF16, M, N, K, 2, splits)[0]["large"] == (K >= 256)


# us measured, the tiles taken / the best of another form: see large_rate in csrc/kernels_gemm.hip.  Weights that no benchmarked model has
@pytest.mark.parametrize("M,N,K,cfg,splits", [(384, 4096, 3072, 5, 4), (1144, 524, 640, 5, 1), (2130, 1096, 640, 5, 1), (440, 12288, 6144, 2, 2),      # 24.3/25.0 11.7/14.2 12.2/14.1 79/87
                                              (700, 12288, 20480, 2, 3), (1711, 5480, 2560, 8, 1), (2700, 7168, 1536, 8, 1), (2120, 640, 4352, 1, 5),  # 300/340 45/50 58/64 26/29
                                              (300, 12288, 1536, 0, 1), (1500, 1536, 512, 5, 1), (900, 5120, 4096, 8, 2)])     # 24/26 11.6/12.9 50/55
def test_models_products_take_the_faster_tiles(M, N, K, cfg, splits):
    assert [(p["cfg"], p["splits"]) for p in exe.exe_op_gemm_model_plan(BF16, M, N, K)] == [(cfg, splits)]


# the same tiles of every form on both sides: 5120 features, N = 4 M, weights of 2^28 elements
@pytest.mark.parametrize("widths,depths,rows", [((5116, 5120), range(512, 20481, 512), range(208, 1281, 16)), ((6396, 6400), range(512, 20481, 512), (1600,)),
                                                ((26212, 26216), (10240,), range(208, 1281, 16))])
def test_four_features_more_do_not_change_the_tiles(widths, depths, rows):
    for K in depths:
        for M in rows:
            a, b = ([(p["rows"], p["cfg"], p["splits"]) for p in exe.exe_op_gemm_model_plan(BF16, M, N, K)] for N in widths)
            assert a == b, (M, K)


@pytest.mark.parametrize("dh", [64, 128])
def test_elements_of_a_head_beyond_32_bits(dh):
    """Extents are as long as the pool: 2^31 elements a head and more."""
    for cap in (8, 1 << 20, (1 << 31) // dh - 8, (1 << 31) // dh, (1 << 32) // dh + 8, (1 << 31) - 8):
        for head in (0, 1, 7, 2 * 96 * 40 - 1):
            for pos in (0, 1, cap - 1):
                for base in (0, 1 << 33):
                    assert exe.exe_op_kv_store_index(base, cap, head, pos, dh) == base + (head * cap + pos) * dh


# us measured, streaming kernel / the best float tile: see F32_STREAM_MARGIN in csrc/kernels_gemm.hip
@pytest.mark.parametrize("M,N,K,route", [(512, 3072, 1024, 1), (1024, 1536, 512, 1), (768, 2048, 512, 1), (1024, 1024, 1024, 1),      # 36/38 20.5/21.4 20.4/21.3 24/29
                                         (1024, 1024, 4096, 1), (2048, 512, 2048, 1), (64, 4096, 1024, 1),                            # 76/105 44/56 9/28
                                         (1152, 1536, 512, 0), (2048, 1024, 1024, 0), (640, 4096, 1024, 0), (512, 4096, 256, 0),      # 24.7/21.6 44/40 64/50 17/13
                                         (2048, 1024, 256, 0), (1024, 4096, 256, 0), (2048, 4096, 1024, 0), (2048, 4096, 256, 0)])    # 17/13 34/20 176/91 60/30
def test_float_products_of_up_to_2048_rows_run_on_the_faster_kernel(M, N, K, route):
    assert exe.exe_op_gemm_plan(F32, M, N, K)["route"] == route
