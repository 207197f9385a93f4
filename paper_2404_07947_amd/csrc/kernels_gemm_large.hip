// GEMM with large tiles (bf16): BM x BN outputs per workgroup, BM 256, 192 or 128 with BN 256, and 256 x 160 and 256 x 128; encode
// batches, and decode batches that split K over workgroups.
//
// What bounds it: MFMA issue and, through the power budget, the clock.  gemm_tile_kernel's loop at this tile size kept the
// matrix pipes busy 66 % of the cycles: its eight waves do the same thing at the same time, so both waves of a SIMD wait
// for the address unit, for LDS and at the barrier together.  Here the waves are two groups of four, one wave of each per
// SIMD, half a phase apart: while one group issues 32 MFMAs back to back, the other fetches the fragments of its next 32
// and starts its share of the loads; a barrier swaps them.  With 16 MFMAs between barriers the hand-over (about 100
// cycles) took back most of the gain; letting the groups' MFMAs overlap at the hand-over, raised wave priority around the
// MFMAs, or loads in front of the fragment reads changed nothing or cost 8 %.
//
// A stage is freed in pieces as it is read (weights and the first half of the activation rows, then the second half), so
// the loads for a piece go out about one and a half k-tiles before it is needed, with the same two stages of LDS.
//
// Outputs in bf16 are turned through LDS as bf16 and leave as whole 128-byte lines, 16 bytes per lane, nontemporal where
// they exceed what a cache would keep for the next kernel: stores of half lines took 400 of 1750 us of the widest launch.
//
// Measured on one MI355X, gemm_tile_kernel 256 x 256 -> this kernel, us per launch (TFLOP/s):
//   16384 x  5120 x  5120   607 (1415) ->  552 (1556)     8192 x 12288 x 12288  1692 (1462) -> 1537 (1610)
//   16384 x 20480 x  5120  2430 (1414) -> 2170 (1584)    16384 x  5120 x 20480  2480 (1385) -> 2254 (1525)
//   12288 x 65536 x  1024  1683 (980)  -> 1224 (1347)     8192 x  3072 x  1024    57 (899)  ->   48 (1085)
// and with the tile height that fills the chip:
//   12288 x  1024 x 16384   396 -> 335 (192 rows)   8192 x 1024 x 1024  36 -> 27, 8192 x 1024 x 4096  92 -> 63 (128 rows)
// Launches of one round or less are bound by what a CU takes in (see large_rate in kernels_gemm.hip); there 256 x 128 and 256 x 160 take
//   512 x 15360 x 5120  84 -> 75 (256 x 128 for 128 x 256)    512 x 20480 x 5120  98 -> 86, 1024 x 20480 x 5120 193 -> 168 (256 x 160 for 192 x 256)
// A third LDS stage where it fits (128 x 256, 256 x 128) gave 2 % and took it back in epilogues of half the rows (where it gives more, 256 x 128
// runs on gemm_tile_kernel's three: runs_large in kernels_gemm.hip); a tile's lines fetched into L2 by
// one of the CUs that share them, some k-tiles ahead, cost as many lines as it saved (3 to 20 % slower).
#include <type_traits>

#include "gemm_tile.h"
#include "kernels.h"

namespace exe {

template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// Outputs of this size and more are stored nontemporal: 12288 x 65536 in bf16 1350 -> 1225 us, 16384 x 5120 557 -> 552;
// of 8192 x 3072 and 8192 x 4096 (50 and 67 MB) the next kernel still finds most in cache, and nothing is gained.
constexpr int64_t NT_BYTES = 96 << 20;
constexpr int LARGE_THREADS = 512;
constexpr int large_lds(int BM, int BN) { return 2 * (BM + BN) * TROW + 8 * 4096; }

// Epilogue for bf16 outputs: a wave's TM x 4 tiles, RJ * 16 rows x 64 features at a time, through its RJ * 2 KB of LDS (16-byte chunk c
// of row r at slot c ^ ((r >> 1) & 7): no bank conflicts either way).  The LDS accesses are inline assembly for the reason
// given at epilogue_tiles.  wide: 0 = rows are 8-byte aligned only, 1 = 16-byte stores, 3 = and nontemporal.
template <int TM, int TN, int MODE, int RJ>
__device__ __forceinline__ void epilogue_rows(const f32x4 (&acc)[TN][TM], unsigned stg, int lane, int row0, int col0, int M, int N,
                                              const bf16_t* __restrict__ bias, float alpha, bf16_t* __restrict__ out, int wide,
                                              const KvStore& kv = KvStore{})
{
    constexpr int CH = TN * 2, RB = CH * 16, NR = (RJ * 16 * CH + 63) / 64;     // 16-byte chunks and bytes of a row, reads of a lane
    constexpr bool SWZ = TN == 4;                    // rows of 160 bytes: chunks in order, read one behind the other
    int lm = lane & 15, lq = lane >> 4;
    f32x4 bv[TN];
#pragma unroll
    for (int i = 0; i < TN; ++i) {
        int n = col0 + i * 16 + lq * 4;
        bv[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (bias && n < N) {
            bf16x4 b = *(const bf16x4*)(bias + n);
#pragma unroll
            for (int e = 0; e < 4; ++e) bv[i][e] = (float)b[e];
        }
    }
    auto turn_row = [&](int p) { return SWZ ? p * 8 + (lane >> 3) : (p * 64 + lane) / CH; };
    auto turn_chunk = [&](int p) { return SWZ ? lane & 7 : (p * 64 + lane) % CH; };
    unsigned waddr[RJ][TN], raddr[NR];
#pragma unroll
    for (int x = 0; x < TN; ++x)
#pragma unroll
        for (int jj = 0; jj < RJ; ++jj) {
            int c = x * 2 + (lq >> 1);
            waddr[jj][x] = stg + (jj * 16 + lm) * RB + ((SWZ ? c ^ lds_swz(jj * 16 + lm) : c) << 4) + (lq & 1) * 8;
        }
#pragma unroll
    for (int p = 0; p < NR; ++p) raddr[p] = stg + turn_row(p) * RB + ((SWZ ? turn_chunk(p) ^ lds_swz(turn_row(p)) : turn_chunk(p)) << 4);
    // 64 features are of one head and all in the cache or none; of 80, each chunk of 8 is
    const bool cached = MODE == EPI_T_KV && col0 + (SWZ ? 0 : TN * 16 - 8) >= kv.first_col;
    KvRows<NR> kr;
#pragma unroll
    for (int jp = 0; jp < TM / RJ; ++jp) {
        if (MODE == EPI_T_KV && cached) kr.load(kv, M, [&](int p) { return row0 + jp * RJ * 16 + turn_row(p); });
#pragma unroll
        for (int jj = 0; jj < RJ; ++jj)
#pragma unroll
            for (int i = 0; i < TN; ++i) {
                f32x4 r = acc[i][jp * RJ + jj] * alpha + bv[i];
                bf16x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = (bf16_t)(MODE == EPI_T_RELU ? act_apply(r[e], 0) : MODE == EPI_T_GELU ? act_apply(r[e], 1) : r[e]);
                asm volatile("ds_write_b64 %0, %1" ::"v"(waddr[jj][i]), "v"(w) : "memory");
            }
        f32x4 v[NR];
        LdsTurn<NR>::read(v, raddr);
#pragma unroll
        for (int p = 0; p < NR; ++p) {
            int m = row0 + jp * RJ * 16 + turn_row(p), n = col0 + turn_chunk(p) * 8;
            if (m >= M || n >= N || turn_row(p) >= RJ * 16) continue;
            bf16_t* o = out + (int64_t)m * N + n;
            if (MODE == EPI_T_KV && cached) {
                if (SWZ) o = (bf16_t*)kv.pool + kr.at(kv, p, col0) + turn_chunk(p) * 8;
                else if (n >= kv.first_col) o = (bf16_t*)kv.pool + kr.at(kv, p, n);
            }
            if (wide & 2) __builtin_nontemporal_store(v[p], (f32x4*)o);
            else if (wide) *(f32x4*)o = v[p];
            else {
                typedef __attribute__((ext_vector_type(2))) float f32x2;
                *(f32x2*)o = f32x2{v[p][0], v[p][1]};
                if (n + 4 < N) *(f32x2*)(o + 4) = f32x2{v[p][2], v[p][3]};
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A stage holds 64 k of [activation rows, half 0 | half 1 | weight rows], 128 bytes a row.  Group g of the waves computes rows
// g * BM/2 .. of the tile: waves of 64 features (BN 256) and all of those rows, or (BN 160, 128) of half the features and 64 rows.  Half h
// of the activations holds the h-th half of every wave's rows.
//
// One k-tile is two phases per group, each a memory step and a compute step, and the groups are one step apart:
//   step     0        1        2        3        4
//   group 0  mem 0    mma 0    mem 1    mma 1    (next k-tile)
//   group 1           mem 0    mma 0    mem 1    mma 1
// mem 0 reads all weight fragments and those of activation half 0, mem 1 those of half 1; either ends with its reads done
// (lgkmcnt 0) in front of the barrier.  Refills, for k-tile kt + 2: the weights in mem 1 of kt (group 1 has read them by
// the end of step 1, group 0 issues in step 2), the activations in mem 0 of kt + 1 (half 1 read by the end of step 3).
// What a phase reads is waited for one phase ahead, by count: every wave issues the same loads, and the barrier makes its
// wait good for all.  Loads of a wave per piece: weights BN / 64 (BN 160: 3 or 2, group 0 or 1), a half of the activations 2 (BM 256),
// 2 or 1 (BM 192: group 0 or 1), 1 (BM 128).
template <int BM, int BN>
__global__ __launch_bounds__(LARGE_THREADS) void gemm_large_kernel(int M, int N, int K, const bf16_t* __restrict__ A,
    const bf16_t* __restrict__ W, const bf16_t* __restrict__ bias, int act, float alpha, int out_mode, void* __restrict__ out,
    float* __restrict__ partial, int tiles_m, int tiles_n, int k_per_split, int n_split, int wide, int lda, int ldw, KvStore kv)
{
    constexpr int NWN = BN == 256 ? 4 : 2, NWR = 4 / NWN;            // waves of a group side by side in the features, and in the rows
    constexpr int WC = BN / NWN, TN = WC / 16;                       // features and 16-feature tiles of a wave
    constexpr int WR = BM / 2 / NWR, TM = WR / 16, TH = TM / 2;      // rows and 16-row tiles of a wave, tiles of one of its halves
    constexpr int QA = WR / 2;                       // rows of a wave in one activation slot
    constexpr int SLOT_A = BM / 2 * TROW;
    constexpr int STAGE = 2 * SLOT_A + BN * TROW;    // [A half 0][A half 1][W]
    constexpr int WP = (BN + 63) / 64;               // 1 KB loads of a wave for the weights of a k-tile, in group 0 and 1
    constexpr int WL0 = WP, WL1 = BN / 64;
    constexpr int AL0 = BM == 128 ? 1 : 2, AL1 = BM == 256 ? 2 : 1;  // and for an activation slot
    constexpr int EN = TN == 4 ? 32 : 16, RJ = TN == 4 ? 2 : 1;      // columns and 16-row tiles that a wave turns through LDS at a time
    extern __shared__ __align__(16) unsigned char lds[];
    int tid = threadIdx.x, lane = tid & 63;
    int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int grp = wave >> 2, wn = wave & (NWN - 1), part = grp * NWR + (wave & 3) / NWN;        // part: the wave's rows

    // Work items are (split, output tile) pairs, mapped as in gemm_tile_kernel: an XCD's 32 workgroups get a patch of 8 x 4
    // tiles.  (4 x 8 is 2 % faster at K = 20480 and 1-3 % slower elsewhere; shifting the patches of the XCDs against each other
    // costs 5 %: they share the weights that the memory-side cache delivers.)
    int total = tiles_m * tiles_n;
    int items = total * n_split;
    auto locate = [&](int v, int& m0, int& n0, int& z) {
        z = v / total;
        int pid = v - z * total;
        int chunk = total / 8;
        if (pid < chunk * 8) pid = (pid % 8) * chunk + pid / 8;
        constexpr int GM = 8;
        int group = pid / (GM * tiles_n);
        int first_m = group * GM;
        int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM;
        int within = pid - group * GM * tiles_n;
        m0 = (first_m + within % gsz) * BM;
        n0 = (within / gsz) * BN;
    };
    auto k_tiles = [&](int z) {
        int kbeg = z * k_per_split;
        int kend = kbeg + k_per_split < K ? kbeg + k_per_split : K;
        return (kend - kbeg) / 64;
    };

    // ---- loader: two k-tiles ahead of the compute steps, across item boundaries; uniform tile origins plus per-lane offsets,
    // rows clamped into the matrices (rows past the edge are never stored).  Inline assembly for the reason given in
    // gemm_tile_kernel.
    unsigned off_a[2][2], off_w[WP];
    const char *base_a, *base_w;
    int ld_v = blockIdx.x, ld_kt = 0, ld_nk = 1;
    int ld_st = 0;
    auto set_src = [&](int v) {
        int m0, n0, z;
        locate(v, m0, n0, z);
        int kbeg = z * k_per_split;
        ld_nk = k_tiles(z);
        base_a = (const char*)(A + (int64_t)m0 * lda + kbeg);
        base_w = (const char*)(W + (int64_t)n0 * ldw + kbeg);
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int p = 0; p < 2; ++p) {
                int s = (p * 8 + wave) * 8 + (lane >> 3);          // row of the slot
                int r = s / QA * WR + h * QA + s % QA;             // row of the tile
                if (m0 + r >= M) r = M - 1 - m0;
                off_a[h][p] = (unsigned)r * (unsigned)(lda * 2) + (((lane & 7) ^ lds_swz(s)) << 4);
            }
#pragma unroll
        for (int p = 0; p < WP; ++p) {
            int s = (p * 8 + wave) * 8 + (lane >> 3), r = s;
            if (n0 + r >= N) r = N - 1 - n0;
            off_w[p] = (unsigned)r * (unsigned)(ldw * 2) + (((lane & 7) ^ lds_swz(s)) << 4);
        }
    };
    set_src(ld_v);
    unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    auto load_to_lds = [&](const char* src, unsigned voff, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
#pragma clang diagnostic pop
    auto load_a = [&](int h) {
        if (EXE_GEMM_ABLATE & 2) return;
        unsigned dst = lds_base + ld_st * STAGE + h * SLOT_A + wave * 1024;
        const char* src = base_a + ld_kt * TROW;
        load_to_lds(src, off_a[h][0], dst);
        if (AL1 == 2 || (AL0 == 2 && grp == 0)) load_to_lds(src, off_a[h][1], dst + 8192);
    };
    auto load_w = [&]() {
        if (EXE_GEMM_ABLATE & 4) return;
        unsigned dst = lds_base + ld_st * STAGE + 2 * SLOT_A + wave * 1024;
        const char* src = base_w + ld_kt * TROW;
#pragma unroll
        for (int p = 0; p < WP; ++p)
            if (p < WL1 || grp == 0) load_to_lds(src, off_w[p], dst + p * 8192);
    };
    // past the last item the last k-tile is loaded again, which keeps the number of loads in flight uniform
    auto advance = [&]() {
        ld_st ^= 1;
        if (ld_kt + 1 < ld_nk) ++ld_kt;
        else if (ld_v + (int)gridDim.x < items) {
            ld_v += gridDim.x;
            ld_kt = 0;
            set_src(ld_v);
        }
    };
    // all but the youngest weight loads of W k-tiles and activation loads of NA slots have landed
    auto wait_loads = [&](auto w, auto na) {
        constexpr int W = decltype(w)::value, NA = decltype(na)::value;
        if (WL0 * W + AL0 * NA == WL1 * W + AL1 * NA || grp == 0) wait_vm<WL0 * W + AL0 * NA>();
        else wait_vm<WL1 * W + AL1 * NA>();
    };
    using C0 = std::integral_constant<int, 0>;
    using C1 = std::integral_constant<int, 1>;
    using C2 = std::integral_constant<int, 2>;
    auto barrier = [&]() { asm volatile("s_barrier" ::: "memory"); };
    auto lgkm0 = [&]() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); };

    f32x4 acc[TN][TM];
    u32x4 fa[TH][2], fw[TN][2];
    int frow = lane & 15, fk = lane >> 4;
    unsigned fo[2];
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fo[ks] = frow * TROW + (((ks * 4 + fk) ^ lds_swz(frow)) << 4);
    auto read_a = [&](int stage, int h, int ks) {
        const unsigned char* s = lds + stage * STAGE + h * SLOT_A + part * QA * TROW;
#pragma unroll
        for (int j = 0; j < TH; ++j) fa[j][ks] = *(const u32x4*)(s + fo[ks] + j * 16 * TROW);
    };
    auto read_w = [&](int stage, int ks) {
        const unsigned char* s = lds + stage * STAGE + 2 * SLOT_A + wn * WC * TROW;
#pragma unroll
        for (int i = 0; i < TN; ++i) fw[i][ks] = *(const u32x4*)(s + fo[ks] + i * 16 * TROW);
    };
#define EXE_SB __builtin_amdgcn_sched_barrier(0)
    auto compute = [&](auto half) {
        constexpr int J0 = decltype(half)::value * TH;
        EXE_SB;
#pragma unroll
        for (int ks = 0; ks < ((EXE_GEMM_ABLATE & 1) ? 0 : 2); ++ks)
#pragma unroll
            for (int i = 0; i < TN; ++i)
#pragma unroll
                for (int j = 0; j < TH; ++j) acc[i][J0 + j] = HalfUnit<bf16_t>::mma(fw[i][ks], fa[j][ks], acc[i][J0 + j]);
        EXE_SB;
        barrier();
        EXE_SB;
    };

    // prologue: k-tile 0 and the weights of k-tile 1; waits for what the first memory step reads
    load_w(); load_a(0); load_a(1); advance();
    load_w();
    wait_loads(C1{}, C1{});
    barrier();
    int st = 0;
    bool first = true;
    for (int v = blockIdx.x; v < items; v += gridDim.x) {
        int m0, n0, z;
        locate(v, m0, n0, z);
        int nk = k_tiles(z);
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if (grp) barrier();                          // the groups part by a step
        for (int kt = 0; kt < nk; ++kt) {
            EXE_SB;
            read_w(st, 0); read_a(st, 0, 0); read_w(st, 1); read_a(st, 0, 1);
            if (kt > 0 || first) {                   // else done before the epilogue of the item before
                load_a(0); load_a(1);
                advance();
                wait_loads(C1{}, C2{});
            }
            lgkm0();
            barrier();
            compute(C0{});
            read_a(st, 1, 0); read_a(st, 1, 1);
            load_w();
            wait_loads(C1{}, C1{});
            lgkm0();
            barrier();
            compute(C1{});
            st ^= 1;
        }
        if (!grp) barrier();                         // and meet again, so that their epilogues run side by side
        first = false;
        // The next item's first k-tile waits for nothing younger than the epilogue's stores until its second phase: the
        // activations of k-tile 1 go out now, and all but those have landed before the first store.
        load_a(0); load_a(1);
        advance();
        wait_loads(C0{}, C2{});
        {
            unsigned stg = lds_base + 2 * STAGE + wave * 4096;
            int row0 = m0 + part * WR, col0 = n0 + wn * WC;
            int el = lane;
            if (TN != 4) asm volatile("" : "+v"(el));        // opaque: held through the loop above, the addresses would spill 11 registers
            if (EXE_GEMM_ABLATE & 32) {            // measurement variant: no epilogue, the accumulators are only kept alive
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j) asm volatile("" ::"v"(acc[i][j]));
            } else if (n_split > 1)
                epilogue_tiles<bf16_t, TM, TN, EN, EPI_PARTIAL>(acc, stg, el, row0, col0, M, N, nullptr, 1.f, partial + (int64_t)z * M * N, nullptr);
            else if (out_mode == OUT_RESID)
                epilogue_tiles<bf16_t, TM, TN, EN, EPI_RESID>(acc, stg, el, row0, col0, M, N, bias, alpha, (float*)out, nullptr);
            else if (out_mode == OUT_F32)
                epilogue_tiles<bf16_t, TM, TN, EN, EPI_F32>(acc, stg, el, row0, col0, M, N, bias, alpha, (float*)out, nullptr);
            else if (kv.pool)
                epilogue_rows<TM, TN, EPI_T_KV, RJ>(acc, stg, el, row0, col0, M, N, bias, alpha, (bf16_t*)out, wide, kv);
            else if (act == 0)
                epilogue_rows<TM, TN, EPI_T_RELU, RJ>(acc, stg, el, row0, col0, M, N, bias, alpha, (bf16_t*)out, wide);
            else if (act == 1)
                epilogue_rows<TM, TN, EPI_T_GELU, RJ>(acc, stg, el, row0, col0, M, N, bias, alpha, (bf16_t*)out, wide);
            else
                epilogue_rows<TM, TN, EPI_T, RJ>(acc, stg, el, row0, col0, M, N, bias, alpha, (bf16_t*)out, wide);
        }
    }
#undef EXE_SB
    wait_vm<0>();     // the loads past the end land before the workgroup's LDS is released
}

template <int BM, int BN>
static hipError_t launch_large(const GemmArgs& a, int k_per_split, int splits, int grid_max, hipStream_t s)
{
    auto kern = gemm_large_kernel<BM, BN>;
    constexpr int lds = large_lds(BM, BN);
    static_assert(lds <= 160 * 1024, "LDS budget");
    static LdsLimit limit[MAX_DEVICES];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
    hipError_t e = limit[dev].raise((const void*)kern, lds);
    if (e != hipSuccess) return e;
    int tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN, items = tm * tn * splits;
    int wide = a.N % 8 == 0 && ((uintptr_t)a.out & 15) == 0 ? (int64_t)a.M * a.N * 2 >= NT_BYTES ? 3 : 1 : 0;
    kern<<<items < grid_max ? items : grid_max, LARGE_THREADS, lds, s>>>(
        a.M, a.N, a.K, (const bf16_t*)a.A, (const bf16_t*)a.W, (const bf16_t*)a.bias, a.act, a.alpha, a.out_mode, a.out, a.workspace, tm,
        tn, k_per_split, splits, wide, a.lda ? a.lda : a.K, a.ldw ? a.ldw : a.K, a.kv ? *a.kv : KvStore{});
    return hipGetLastError();
}

hipError_t launch_gemm_large(const GemmArgs& a, int bm, int bn, int k_per_split, int splits, int grid_max, hipStream_t s)
{
    return bn == 128 ? launch_large<256, 128>(a, k_per_split, splits, grid_max, s)
         : bn == 160 ? launch_large<256, 160>(a, k_per_split, splits, grid_max, s)
         : bm == 256 ? launch_large<256, 256>(a, k_per_split, splits, grid_max, s)
         : bm == 192 ? launch_large<192, 256>(a, k_per_split, splits, grid_max, s)
                     : launch_large<128, 256>(a, k_per_split, splits, grid_max, s);
}

}  // namespace exe
