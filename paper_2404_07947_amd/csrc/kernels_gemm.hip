// GEMM kernels for the projections of a Transformer layer: out = epilogue(alpha * A[M,K] . W[N,K]^T + bias).
//
//  * gemm_tile_kernel    MFMA 16x16x32, bf16.  Macro tiles (BM x 256 or BM x 128, 128 bytes of K
//                        per LDS stage) filled by direct global->LDS loads into a ring of stages; software-pipelined
//                        fragment fetch; optional split-K into float partials, finished by splitk_reduce_kernel.
//  * gemm_large_kernel   (kernels_gemm_large.hip) bf16, tiles of 128 rows and 128 features or more, K of 256 and more: encode,
//                        and decode batches of 100 rows and more.
//  * gemm_f32_kernel     (kernels_gemm_f32.hip) float, many rows.
//  * gemm_stream_kernel  (kernels_gemm_stream.hip) few rows: streams the weights, the waves of a workgroup split K.
//  * gemm_generic_kernel float or bf16 inputs, plain FMA in float, any shape (depths and widths the others do not take).
//
// Both A and W are K-contiguous, so both MFMA operands are 16-byte vectors along K.  The MFMA "A" operand
// is fed with weight rows and the "B" operand with activation rows: the accumulator then holds 4
// consecutive output features per lane, which makes the epilogue's loads and stores 8/16-byte vectors.
#include <algorithm>
#include <stdlib.h>

#include <mutex>
#include <type_traits>
#include <unordered_map>

#include "gemm_tile.h"
#include "kernels.h"

// gemm_tile_kernel: sub-step of a k-tile (8 MFMAs each) at which the second of the four parts of the next stage's loads is issued;
// the third and fourth follow one sub-step apart.  0 in the library; other values build measurement variants
// (-1 issues the second part with the first, behind the barrier).
#ifndef EXE_GEMM_ISSUE_AT
#define EXE_GEMM_ISSUE_AT 0
#endif

namespace exe {

// Columns that a wave turns through LDS at a time in the epilogue: 32 (4 KB per wave) where the stages leave
// room within the 160 KB of a CU, else 16 (2 KB per wave).
constexpr int epilogue_cols(int BM, int BN, int WM, int WN, int ST)
{
    return ST * (BM + BN) * TROW + (BM / WM) * (BN / WN) * 4096 <= 160 * 1024 ? 32 : 16;
}

// ---------------------------------------------------------------- tile kernel
// Tiles are filled with direct global->LDS loads (no staging registers): one wave-wide 16-byte load
// writes 1 KB of consecutive tile rows, lane l landing at byte 16*l.  The swizzle is therefore applied on
// the global side: lane l fetches chunk (l % 8) ^ swz(row) of row l / 8.
//
// ST LDS stages of 64 k form a ring: while k-tile kt is multiplied, k-tiles kt+1 .. kt+ST-1 are in flight.
// Inside a k-tile the loop is software-pipelined over sub-steps (32 k x 32 rows of the wave's tile): the operand
// fragments of sub-step s+1 are fetched from LDS before the MFMAs of sub-step s are issued.  The one barrier per
// k-tile sits in front of the MFMAs of its last sub-step: behind it every wave has finished reading the current
// stage and k-tile kt+1 has landed, so the loads of k-tile kt+ST go into the stage just vacated and the first
// fragments of k-tile kt+1 are fetched while the last MFMAs of k-tile kt execute.
//
// The MFMA is the 16x16x32 one (4 passes).  Measured on MI355X: while a SIMD executes 32x32x16 MFMAs (8 passes)
// back to back, vector memory instructions of the waves on it are hardly issued at all (a loader wave beside an
// MFMA wave ran 20x slower), so the tile loads and the MFMAs of a k-tile ran one after the other; beside
// back-to-back 16x16x32 MFMAs the same loads run at 92 % of their stand-alone rate, at an equal MFMA rate.
//
// Workgroups are persistent (one per CU) and the loader runs ahead across items, so that a tile's epilogue and
// the first loads of the next tile overlap.  Split-K (n_split > 1): every item writes its float partial tile;
// splitk_reduce_kernel finishes.
template <typename T, int BM, int BN, int WM, int WN, int ST>
__global__ __launch_bounds__((BM / WM) * (BN / WN) * 64) void gemm_tile_kernel(
    int M, int N, int K, const T* __restrict__ A, const T* __restrict__ W, const T* __restrict__ bias, int act, float alpha, int out_mode, void* __restrict__ out, float* __restrict__ partial, int tiles_m, int tiles_n,
    int k_per_split, int n_split, int flags, int lda, int ldw)
{
    // flags: bit 0 = spread the loads of a k-tile over the MFMAs (see below); bit 1 = the weights are read once
    // (a single row of output tiles): their loads are marked nontemporal so that they do not displace A in L2
    const int spread = flags & 1;
    const bool w_once = (flags & 2) != 0;
    constexpr int NW = (BM / WM) * (BN / WN);
    constexpr int TM = WM / 16, TN = WN / 16;       // 16x16 accumulator tiles of a wave: TM along rows, TN along features
    constexpr int MH = TM > 2 ? TM / 2 : 1;         // row parts of the wave's tile, one per sub-step
    constexpr int TMH = TM / MH;
    constexpr int NS = 2 * MH;                      // sub-steps per k-tile
    constexpr int A_PASSES = BM / 8 / NW, B_PASSES = BN / 8 / NW;   // 1 KB wave-loads per wave per stage
    // wave-loads a wave issues per k-tile (all of them, unless a measurement variant drops an operand's)
    constexpr int LPT = ((EXE_GEMM_ABLATE & 2) ? 0 : A_PASSES) + ((EXE_GEMM_ABLATE & 4) ? 0 : B_PASSES);
    constexpr int LPX = A_PASSES + B_PASSES;      // positions of the issue sequence: A passes, then W passes
    static_assert((BM / 8) % NW == 0 && (BN / 8) % NW == 0, "tile/waves mismatch");
    static_assert(LPT * (ST - 1) <= 63, "vmcnt range");
    extern __shared__ __align__(16) unsigned char lds[];
    constexpr int STAGE = (BM + BN) * TROW;        // bytes per LDS stage: A tile then W tile
    constexpr int TBK = tbk<T>();
    constexpr unsigned ESZ = sizeof(T);
    constexpr int EN = epilogue_cols(BM, BN, WM, WN, ST);

    // Work items are (split, output tile) pairs, numbered split-major.  The workgroups are persistent: workgroup b
    // takes items b, b + gridDim.x, ...  Item -> tile: consecutive item numbers on one XCD (workgroups are
    // dispatched round-robin over 8 XCDs and gridDim.x is a multiple of 8 whenever a workgroup takes more than
    // one item) get a GM x (32/GM) patch of tiles so that the XCD's L2 sees each A and W tile a few times only.
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
        return (kend - kbeg) / TBK;
    };

    int tid = threadIdx.x, lane = tid & 63;
    int wave = __builtin_amdgcn_readfirstlane(tid >> 6);      // wave-uniform: keeps what derives from it in SGPRs
    int wm = wave % (BM / WM), wn = wave / (BM / WM);

    // ---- loader: runs ST k-tiles ahead of the MFMA loop, across item boundaries.  The source of a wave-load is a
    // uniform tile origin plus a per-lane byte offset (row clamped into the matrix; rows past the edge are never
    // stored), which keeps the addresses in 8 registers.
    unsigned off_a[A_PASSES], off_w[B_PASSES];
    const char *base_a, *base_w;
    int ld_v = blockIdx.x, ld_kt = 0, ld_nk = 1;
    auto set_src = [&](int v) {
        int m0, n0, z;
        locate(v, m0, n0, z);
        int kbeg = z * k_per_split;
        ld_nk = k_tiles(z);
        base_a = (const char*)(A + (int64_t)m0 * lda + kbeg);
        base_w = (const char*)(W + (int64_t)n0 * ldw + kbeg);
#pragma unroll
        for (int p = 0; p < A_PASSES; ++p) {
            int rl = (p * NW + wave) * 8 + (lane >> 3);
            int r = m0 + rl < M ? rl : M - 1 - m0;
            off_a[p] = (unsigned)r * (unsigned)lda * ESZ + (((lane & 7) ^ lds_swz(rl)) << 4);
        }
#pragma unroll
        for (int p = 0; p < B_PASSES; ++p) {
            int rl = (p * NW + wave) * 8 + (lane >> 3);
            int r = n0 + rl < N ? rl : N - 1 - n0;
            off_w[p] = (unsigned)r * (unsigned)ldw * ESZ + (((lane & 7) ^ lds_swz(rl)) << 4);
        }
    };
    set_src(ld_v);
    // issues wave-loads X0 .. X1-1 (A passes first, then W passes) of the loader's current k-tile into `stage`.
    // The load is written as inline assembly on purpose: the compiler assumes that any later DS read may alias
    // the destination of a direct-to-LDS load it knows of, and puts a vmcnt(0) in front of the fragment reads,
    // which empties the ring of stages at every k-tile.  Completion is tracked by the explicit waits below.
    unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds;
    // (m0, the LDS destination, is a reserved register: naming it as clobbered draws a warning, but keeps the
    // compiler from merging its own m0 set-ups across the statement)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    auto load_to_lds = [&](const char* src, unsigned voff, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
    auto load_to_lds_nt = [&](const char* src, unsigned voff, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
#pragma clang diagnostic pop
    auto issue_range = [&](int stage, auto x0, auto x1) {
        unsigned base = lds_base + stage * STAGE + wave * 1024;
        const char* ka = base_a + ld_kt * TROW;
        const char* kw = base_w + ld_kt * TROW;
#pragma unroll
        for (int x = decltype(x0)::value; x < decltype(x1)::value; ++x) {
            if ((EXE_GEMM_ABLATE & 2) && x < A_PASSES) continue;
            if ((EXE_GEMM_ABLATE & 4) && x >= A_PASSES) continue;
            if (x < A_PASSES) load_to_lds(ka, off_a[x], base + x * NW * 1024);
            else if (w_once) load_to_lds_nt(kw, off_w[x - A_PASSES], base + BM * TROW + (x - A_PASSES) * NW * 1024);
            else load_to_lds(kw, off_w[x - A_PASSES], base + BM * TROW + (x - A_PASSES) * NW * 1024);
        }
    };
    // moves the loader to the next k-tile; past the last item the last k-tile is loaded again, which keeps the
    // number of loads in flight uniform
    auto advance = [&]() {
        if (ld_kt + 1 < ld_nk) ++ld_kt;
        else if (ld_v + (int)gridDim.x < items) {
            ld_v += gridDim.x;
            ld_kt = 0;
            set_src(ld_v);
        }
    };
    // A k-tile's loads are issued in four parts spread over 24 MFMAs: a burst of all of them fills the queue of
    // the CU's address unit, and a wave waiting to issue a load issues no MFMA either.
    // (`spread` = 0 issues them all at once behind the barrier.)
    constexpr int IA = EXE_GEMM_ISSUE_AT > NS - 4 ? NS - 4 : EXE_GEMM_ISSUE_AT;     // all four parts go out inside the k-tile
    constexpr int Q1 = LPX / 4, Q2 = LPX / 2, Q3 = LPX * 3 / 4;
    using X0 = std::integral_constant<int, 0>;
    using X1 = std::integral_constant<int, Q1>;
    using X2 = std::integral_constant<int, Q2>;
    using X3 = std::integral_constant<int, Q3>;
    using X4 = std::integral_constant<int, LPX>;

    // MFMA operands: lane l holds 16-byte chunk 4*ks + l/16 of stage row l%16: the 8 k-values 8*(l/16) .. +7 of a 32-k step.
    // The W fragments of a step are kept for all its row parts.
    f32x4 acc[TN][TM];
    int frow = lane & 15, fk = lane >> 4;
    u32x4 fa[2][TMH], fw[2][TN];
    // fragments of sub-step s of the k-tile in `stage`: activation rows of its row part, and (first row part of a
    // 32-k step only) the weight rows
    auto fetch = [&](int stage, int s) {
        const unsigned char* sa = lds + stage * STAGE;
        const unsigned char* sw = sa + BM * TROW;
        int ks = s / MH, mh = s % MH;
#pragma unroll
        for (int j = 0; j < TMH; ++j)
            fa[s & 1][j] = *(const u32x4*)(sa + lds_off(wm * WM + (mh * TMH + j) * 16 + frow, ks * 4 + fk));
        if (mh == 0) {
#pragma unroll
            for (int i = 0; i < TN; ++i) fw[ks & 1][i] = *(const u32x4*)(sw + lds_off(wn * WN + i * 16 + frow, ks * 4 + fk));
        }
    };
    // the MFMAs of sub-step s in two halves, so that the next sub-step's fragment fetch can be issued between them
    auto mma = [&](int s, int half) {
        constexpr int NM = TN * TMH;
        int ks = s / MH, mh = s % MH;
        if (EXE_GEMM_ABLATE & 1) return;
#pragma unroll
        for (int x = 0; x < NM; ++x) {
            if ((x < NM / 2) != (half == 0)) continue;
            int i = x / TMH, j = x % TMH;
            acc[i][mh * TMH + j] = HalfUnit<T>::mma(fw[ks & 1][i], fa[s & 1][j], acc[i][mh * TMH + j]);
        }
    };
#define EXE_SB __builtin_amdgcn_sched_barrier(0)

    // prologue: the first ST k-tiles go to stages 0 .. ST-1; wait for the first only
#pragma unroll
    for (int t = 0; t < ST; ++t) {
        issue_range(t, X0{}, X4{});
        advance();
    }
    wait_cnt<LPT*(ST - 1), 15>();
    __syncthreads();
    fetch(0, 0);
    int st = 0, fill_st = 0;
    bool pend = false;        // parts 2 .. 4 of the k-tile going into stage fill_st are still to be issued
    for (int v = blockIdx.x; v < items; v += gridDim.x) {
        int m0, n0, z;
        locate(v, m0, n0, z);
        int nk = k_tiles(z);
#pragma unroll
        for (int i = 0; i < TN; ++i)
#pragma unroll
            for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        for (int kt = 0; kt < nk; ++kt) {
            int nst = st + 1 == ST ? 0 : st + 1;
            // Every sub-step but the last: the fetch of the following sub-step's fragments, then the MFMAs (a full
            // sub-step of MFMAs between a fetch and its use).  The first three also issue the rest of the loads
            // whose first part went out behind the previous barrier.
            if constexpr (NS >= 4) {
#pragma unroll
                for (int s = 0; s < NS - 1; ++s) {
                    fetch(st, s + 1);
                    if (s == IA && pend) issue_range(fill_st, X1{}, X2{});
                    if (s == IA + 1 && pend) issue_range(fill_st, X2{}, X3{});
                    if (s == IA + 2 && pend) {
                        issue_range(fill_st, X3{}, X4{});
                        advance();
                    }
                    EXE_SB; mma(s, 0); mma(s, 1); EXE_SB;
                }
            } else {
                fetch(st, 1);
                if (pend) issue_range(fill_st, X1{}, X2{});
                EXE_SB; mma(0, 0); EXE_SB;
                if (pend) issue_range(fill_st, X2{}, X3{});
                EXE_SB; mma(0, 1); EXE_SB;
                if (pend) {
                    issue_range(fill_st, X3{}, X4{});
                    advance();
                }
            }
            // last sub-step of the k-tile.  Its fragments were the last reads of this stage: once they have
            // returned (lgkmcnt 0) and the following k-tile has landed (all but the ST-2 most recent k-tiles'
            // loads), synchronise, start refilling the stage just vacated and fetch the first fragments of the
            // following k-tile of this item behind the barrier, a full sub-step ahead of their use.
            wait_cnt<LPT*(ST - 2), 0>();
            __syncthreads();
            issue_range(st, X0{}, X1{});
            if (IA < 0 && NS >= 4 && spread) issue_range(st, X1{}, X2{});
            if (spread) {
                fill_st = st;
                pend = true;
            } else {
                issue_range(st, X1{}, X4{});
                advance();
            }
            if (kt + 1 < nk) fetch(nst, 0);
            EXE_SB; mma(NS - 1, 0); mma(NS - 1, 1); EXE_SB;
            st = nst;
        }
        // Epilogue; its stores drain while the next item's first k-tiles are multiplied.
        {
            unsigned stg = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds + ST * STAGE + wave * (EN * 128);
            int row0 = m0 + wm * WM, col0 = n0 + wn * WN;
            if (EXE_GEMM_ABLATE & 32) {            // measurement variant: no epilogue, the accumulators are only kept alive
#pragma unroll
                for (int i = 0; i < TN; ++i)
#pragma unroll
                    for (int j = 0; j < TM; ++j) asm volatile("" ::"v"(acc[i][j]));
            } else if (n_split > 1)
                epilogue_tiles<T, TM, TN, EN, EPI_PARTIAL>(acc, stg, lane, row0, col0, M, N, nullptr, 1.f, partial + (int64_t)z * M * N, nullptr);
            else if (out_mode == OUT_RESID)
                epilogue_tiles<T, TM, TN, EN, EPI_RESID>(acc, stg, lane, row0, col0, M, N, bias, alpha, (float*)out, nullptr);
            else if (out_mode == OUT_F32)
                epilogue_tiles<T, TM, TN, EN, EPI_F32>(acc, stg, lane, row0, col0, M, N, bias, alpha, (float*)out, nullptr);
            else if (act == 0)
                epilogue_tiles<T, TM, TN, EN, EPI_T_RELU>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (T*)out);
            else if (act == 1)
                epilogue_tiles<T, TM, TN, EN, EPI_T_GELU>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (T*)out);
            else
                epilogue_tiles<T, TM, TN, EN, EPI_T>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (T*)out);
        }
        // first fragments of the next item (not held across the epilogue: it needs the registers)
        if (v + (int)gridDim.x < items) fetch(st, 0);
    }
#undef EXE_SB
    wait_cnt<0, 15>();     // drain the tail loads before the workgroup's LDS is released
}

// Sums the split-K partials in split order (deterministic) and applies the epilogue.  (A reduction fused
// into the GEMM through arrival counters was measured 3x slower: the device-scope fences it needs write
// back and invalidate the L2 for every workgroup.)
// What bounds it: the partial sums, read once, most of them from cache.  One index over the rows' groups of 4 columns, of 32 bits: its division by
// the row's groups runs under the loads, three parts of which are in flight.  us of this kernel with an index of 64 bits, with a row per grid row (in
// workgroups of 1024 columns) and so: 4096 x 1028 in 4 parts 13.5, 19.7, 12.6, 4096 x 3076 in 2 21.7, 24.9, 20.8, 512 x 5120 in 3 5.7, 5.4, 5.3, 1000 x 3072 in
// 2 4.5, 4.5, 4.5; a wave per 256 columns of a row is between them.  Two groups a thread, or nontemporal loads, took 1 to 4 % more with the product in front.
constexpr int REDUCE_THREADS = 256;
constexpr int64_t REDUCE_QUADS = (int64_t)1 << 31;       // of a launch
template <typename T>
__global__ __launch_bounds__(REDUCE_THREADS) void splitk_reduce_kernel(unsigned quads, unsigned row_quads, int64_t slice, int S, const float* __restrict__ partial,
                                                                       const T* __restrict__ bias, int act, float alpha, int out_mode,
                                                                       void* __restrict__ out)
{
    const unsigned q = blockIdx.x * REDUCE_THREADS + threadIdx.x;
    if (q >= quads) return;
    const float* p = partial + (int64_t)q * 4;
    f32x4 v = *(const f32x4*)p;
    for (int s = 1; s < S; s += 3) {
        f32x4 t[3];
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (s + j < S) t[j] = *(const f32x4*)(p + (s + j) * slice);
#pragma unroll
        for (int j = 0; j < 3; ++j)
            if (s + j < S) v += t[j];
    }
    const unsigned m = q / row_quads;
    epilogue_store4<T>(v, (int)m, (int)(q - m * row_quads) * 4, (int)row_quads * 4, bias, act, alpha, out_mode, out);
}

// ---------------------------------------------------------------- generic kernel (float math, any shape)
template <typename T>
__global__ __launch_bounds__(256) void gemm_generic_kernel(int M, int N, int K, const T* __restrict__ A,
                                                           const T* __restrict__ W, const T* __restrict__ bias,
                                                           int act, float alpha, int out_mode, void* __restrict__ out)
{
    constexpr int TS = 64, KS = 16;
    __shared__ float sa[KS][TS + 1], sw[KS][TS + 1];
    int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    int m0 = blockIdx.y * TS, n0 = blockIdx.x * TS;
    float acc[4][4] = {};
    for (int k0 = 0; k0 < K; k0 += KS) {
        for (int i = threadIdx.x; i < TS * KS; i += 256) {
            int r = i / KS, k = i % KS;
            sa[k][r] = (m0 + r < M && k0 + k < K) ? to_f32(A[(int64_t)(m0 + r) * K + k0 + k]) : 0.f;
            sw[k][r] = (n0 + r < N && k0 + k < K) ? to_f32(W[(int64_t)(n0 + r) * K + k0 + k]) : 0.f;
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            float a[4], w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) { a[i] = sa[k][ty * 4 + i]; w[i] = sw[k][tx * 4 + i]; }
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
        }
        __syncthreads();
    }
    for (int i = 0; i < 4; ++i) {
        int m = m0 + ty * 4 + i;
        if (m >= M) continue;
        for (int j = 0; j < 4; ++j) {
            int n = n0 + tx * 4 + j;
            if (n >= N) continue;
            float r = acc[i][j] * alpha + (bias ? to_f32(bias[n]) : 0.f);
            int64_t o = (int64_t)m * N + n;
            if (out_mode == OUT_T) ((T*)out)[o] = from_f32<T>(act_apply(r, act));
            else if (out_mode == OUT_RESID) ((float*)out)[o] += r;
            else ((float*)out)[o] = r;
        }
    }
}

// ---------------------------------------------------------------- host-side routing
// Tile configurations.  Four have BN = 256 (the weight share of the LDS fill traffic is BN / (BM + BN), which is what a
// weight-streaming decode GEMM wants large); 64x128, 128x128 and 256x128 halve BN for matrices with few output features,
// where more tiles beat deeper split-K.  The BN = 256 shapes of 128 and more rows run on gemm_large_kernel if K allows, 256x128 on
// either (runs_large), the others on gemm_tile_kernel.  192x256 and 256x160 run on gemm_large_kernel only.
enum Cfg { C64x256 = 0, C128x256, C256x256, C64x128, C128x128, C256x128, C192x256, F64x64, C256x160, N_CFG };      // F64x64: a float tile only
struct CfgInfo { int bm, bn; };
static const CfgInfo CFG[N_CFG] = {{64, 256}, {128, 256}, {256, 256}, {64, 128}, {128, 128}, {256, 128}, {192, 256}, {64, 64}, {256, 160}};

// the shallowest depth of gemm_large_kernel (its start and end take a few k-tiles' time)
static bool is_large(int cfg) { return cfg == C256x256 || cfg == C128x256 || cfg == C192x256 || cfg == C256x128 || cfg == C256x160; }
static bool only_large(int cfg) { return cfg == C192x256 || cfg == C256x160; }
constexpr int LARGE_MIN_K = 256;

// Whether a launch of a configuration runs on gemm_large_kernel.  256 x 128 has a third LDS stage in gemm_tile_kernel, which is the better
// one where lines come late: weights that do not stay in cache, read by few row tiles at once, or parts so deep that the tiles that
// share lines drift apart.  us of gemm_tile_kernel / gemm_large_kernel on either side of the line, whole sums: 256 x 24576, K 3072 51 / 51,
// K 4096 64 / 65, K 6144 99 / 107, 512 x 16384, K 6144 94 / 94, K 12288 188 / 218, 768 x 9216, K 11008 153 / 150, 1024 x 16384, K 12288 342 / 324, K 14336 402 / 439;
// in parts: 256 x 9216, K 4096 in 3 36.7 / 35.5, 256 x 8192, K 8192 in 4 48 / 51, 512 x 5120, K 12288 in 3 75 / 73, 512 x 13824, K 14336 in 2 217 / 231.
// Of 3469 launches of up to 1024 rows gemm_large_kernel alone takes 0.986 of gemm_tile_kernel's time on average and 1.26 at most, by this
// line 0.977 and 1.08.  Beyond them it takes 0.960.
static bool runs_large(int cfg, int M, int N, int K, int splits)
{
    if (!is_large(cfg) || K < LARGE_MIN_K) return false;
    if (cfg != C256x128 || M > 1024) return true;
    const int rows = (M + 255) / 256;
    return splits == 1 ? K < std::min(4096 * rows, 14336) : (int64_t)N * K < (int64_t)std::min(40 * rows, 96) << 20;
}

static int k_tile(int dtype) { return dtype == DT_F32 ? tbk<float>() : tbk<bf16_t>(); }

// route: 0 tile kernel, 1 streaming kernel (then `stream` says how), 2 generic kernel
struct Plan { int route; int cfg; int splits; int k_per_split; int tiles; int spread; double cost; StreamPlan stream; };

static int env_int(const char* name, int dflt)
{
    const char* v = getenv(name);
    return v ? atoi(v) : dflt;
}

// Tuning knobs for sweeps and debugging, read from the environment once per process: EXE_GEMM_CFG forces a tile
// configuration, EXE_GEMM_SPLIT a split count, EXE_GEMM_SPREAD the load issue pattern, EXE_GEMM_NT the
// nontemporal weight loads, EXE_GEMM_GRID the number of persistent workgroups.
struct Knobs { int cfg, split, spread, nt, grid; };
static const Knobs& knobs()
{
    static const Knobs k{env_int("EXE_GEMM_CFG", -1), env_int("EXE_GEMM_SPLIT", 0), env_int("EXE_GEMM_SPREAD", -1),
                         env_int("EXE_GEMM_NT", -1), env_int("EXE_GEMM_GRID", 0)};
    return k;
}

// Cost model behind the choice of tile shape and split count: a workgroup's time is the larger of its LDS-fill traffic and
// its MFMA work, in rounds of one workgroup per CU; the whole launch cannot beat streaming W once from HBM; split-K adds the
// float partials' round trip and a second launch (`defer`: the next kernel of the residual stream adds them up, see
// norm_kernel).
//
// Two sets of rates.  A model's launches (`model`): fitted to 2800 launches on MI355X, 13 row counts from 24 to 2048 x 11
// weight shapes of 1024 to 49152 features, six tile shapes x 1..8 splits, weights from HBM; those of 256x128 and 256x160 afterwards
// to 26100 launches of 2950 shapes, rows 193 to 16384, features 500 to 65536, depths 512 to 20480 (a sixteenth of the shapes at weights of the
// models that the benchmarks name): there the picks take 0.9 % more than the best measured choice on average (without the two 1.8 %; at up to
// 3000 features 1.8 and 2.2 %, wider 0.5 and 1.7 %), 21 % at worst.  On 900 other shapes of these ranges the launches as planned take 0.989 of the time that they
// take without the two, 1.10 at most.
// gemm_large_kernel is priced by its time per k-tile and per tile (large_rate), 16 % more when every CU runs it: the clock falls.  Up to 192
// rows, where the estimate also has to compare with the streaming kernel's, the rates of an earlier fit stay (within 2 % of
// the best choice on average), and so they do for exe_op_gemm's launches up to 1024 rows: its callers have been given these
// plans' workspace sizes.
struct Rates { double fill, mfma, hbm, partial, reduce; };
static const Rates MODEL_RATES{44e9, 3.5e12, 6.5e12, 5.3e12, 4.5e-6}, OP_RATES{35e9, 3.5e12, 5.5e12, 3e12, 1e-6};

// Seconds per k-tile and per tile.  What a CU takes in is bound by the lines that it has in flight, whatever the instructions, and a line
// from HBM takes about twice as long as one from L2.  So the shapes that read fewer weights per activation, 256 x 128 and 256 x 160, gain the
// more, the more of the lines are weights, which come from memory.  Of 2600 pairs of 256 x 128 and 128 x 256, of equal area and the same parts, the
// former takes 0.94 to 0.97 of the latter's time where N is 4 M and more (512 x 15360, K 5120 74 / 84 us), 1.00 where they are equal, and in
// parts 1.03 to 1.06 where M is 2 N and more (1024 x 1024, K 16384 in 8 54 / 46): their prices follow M / (M + N).  That of 256 x 160 follows the
// weights' size besides, without which it was 0.93 of the time at 0.5 GB and 0.87 at 1 GB.  256 x 160 also fits widths that leave the others'
// last round half empty: 512 x 20480, K 5120 86 (192 x 256 98), 1024 x 20480 168 (193).
struct LargeRate { double per, fixed; };
static LargeRate large_rate(int cfg, int M, int N, int K)
{
    const double share = M / ((double)M + N), weights = (double)N * K;
    switch (cfg) {
        case C128x256: return {0.80e-6, 3e-6};
        case C256x128: return {0.76e-6 * (1 + 0.25 * share), 2e-6};
        case C256x160: return {0.78e-6 * (1 + 0.25 * share) * (1 + 0.3 * weights / (weights + (1 << 28))), 3.6e-6};
        case C192x256: return {0.93e-6, 4.5e-6};
        default: return {1.03e-6, 5e-6};
    }
}

static double split_cost(int splits, int M, int N, bool defer, const Rates& r)
{
    return defer ? 2.0 * splits * M * N * 4 / 8e12 - 1e-6 : 2.0 * splits * M * N * 4 / r.partial + r.reduce;
}

static double plan_cost(int dtype, int cfg, int splits, int M, int N, int K, bool defer, bool model)
{
    if (dtype == DT_F32) return gemm_f32_cost(M, N, K);
    int bm = CFG[cfg].bm, bn = CFG[cfg].bn, bk = k_tile(dtype), esz = TROW / bk;
    const Rates& r = model ? MODEL_RATES : OP_RATES;
    int64_t tiles = (int64_t)((M + bm - 1) / bm) * ((N + bn - 1) / bn);
    int64_t wgs = tiles * splits;
    double rounds = (double)((wgs + 255) / 256);
    double ktiles = (double)((K / bk + splits - 1) / splits);
    double t;
    if (model && is_large(cfg)) {
        double busy = wgs / rounds / 256;
        const LargeRate lr = large_rate(cfg, M, N, K);
        t = rounds * (ktiles * lr.per * (1.0 + 0.16 * busy) + lr.fixed);
    } else {
        double fill = ktiles * (bm + bn) * TROW / r.fill;
        double mfma = ktiles * 2.0 * bm * bn * bk / (cfg == C128x256 ? 2.8e12 : r.mfma);
        t = rounds * (fill > mfma ? fill : mfma);
    }
    double hbm = (double)N * K * esz / r.hbm;
    if (t < hbm) t = hbm;
    t += 4e-6;
    if (splits > 1) t += split_cost(splits, M, N, defer, r);
    return t;
}

// Split-K over `s` parts (bf16): every part but the last takes ceil(k-tiles / s) k-tiles, the last one the rest, which
// must be at least 4 k-tiles.  Float is not split: its callers need no workspace, and the few-row shapes that would
// want it run on the streaming kernel.
static int split_k_tiles(int dtype, int K, int s) { return (K / k_tile(dtype) + s - 1) / s; }
static bool split_ok(int dtype, int K, int s)
{
    if (s == 1) return true;
    if (dtype == DT_F32) return false;
    int per = split_k_tiles(dtype, K, s), last = K / k_tile(dtype) - per * (s - 1);
    return per >= 4 && last >= 4;
}

// The streaming kernel is taken when its estimate is clearly below the tile kernel's (both are within 10-20 %): the tile
// kernel's is a few per cent high where both stream from HBM.
constexpr double STREAM_MARGIN = 0.92;
// Float: both estimates are within 2 to 4 %, and the streaming kernel served these shapes before the float tiles were worth it, so
// that near the line it stays.  Of 210 launches of up to 2048 rows (the weights named at gemm_f32_tile) the kernel taken is within 0.2 % of the faster
// one on average, 4 % at worst.  us, streaming / the best tile, on either side of the line:
//    512 x 3072, K 1024 36.4 / 38.2    1024 x 1536, K 512 20.5 / 21.4    768 x 2048, K 512 20.4 / 21.3    1024 x 1024, K 1024 23.5 / 29.4
//    640 x 3072, K 1024 43.9 / 39.6    1152 x 1536, K 512 24.7 / 21.6   1024 x 2048, K 512 26.1 / 22.2   2048 x 1024, K 1024 44.3 / 39.8
//    640 x 4096, K 1024 63.6 / 49.5     512 x 4096, K 256 17.2 / 13.4   1024 x 4096, K 256 33.7 / 19.8   2048 x 4096, K 256 60.4 / 30.0
constexpr double F32_STREAM_MARGIN = 1.08;

constexpr int64_t MANY_ROWS_PARTIALS = 128 << 20;
constexpr int OP_RATE_ROWS = 192;

struct PlanKey {
    int M, N, K, flags;
    bool operator==(const PlanKey& o) const { return M == o.M && N == o.N && K == o.K && flags == o.flags; }
};
struct PlanKeyHash {
    size_t operator()(const PlanKey& k) const
    {
        uint64_t h = (((uint64_t)k.M << 32) ^ (uint64_t)k.N) * 0x9e3779b97f4a7c15ull ^ (((uint64_t)k.K << 3) + k.flags);
        h *= 0x9e3779b97f4a7c15ull;
        return (size_t)(h ^ h >> 32);
    }
};

// mode: what the caller allows (GemmMode)
static Plan make_plan(int dtype, int M, int N, int K, int mode)
{
    Plan p{2, 0, 1, K, 0, 0, 0.0, StreamPlan{}};
    if (N % 4 != 0 || K % k_tile(dtype) != 0 || M < 1) return p;
    // the MFMA kernels address the rows of a tile by 32-bit byte offsets, in float up to 128 rows
    if (dtype == DT_F32 && (int64_t)K * 128 * (int)sizeof(float) >= ((int64_t)1 << 32)) return p;
    p.route = 0;
    p.cfg = dtype == DT_F32 ? C64x128 : C256x256;
    // the model's choice per shape is remembered (a decode iteration asks for the same few shapes 4 times per layer)
    struct Choice { int cfg, splits; double cost; StreamPlan stream; };
    thread_local std::unordered_map<PlanKey, Choice, PlanKeyHash> memo;
    const PlanKey key{M, N, K, mode | (dtype == DT_F32 ? 4 : 0)};
    auto hit = memo.find(key);
    if (hit != memo.end()) {
        p.cfg = hit->second.cfg;
        p.splits = hit->second.splits;
        p.cost = hit->second.cost;
        p.stream = hit->second.stream;
    } else {
        // Beyond 1024 rows a launch has many tiles and only the large shapes are worth a look; split-K still pays where they
        // leave most of the chip idle (1500 x 1024, K 16384: 239 us in 24 tiles, 60 us in six parts), with partial sums
        // bounded, and for a model's launches only (others would have to bring a workspace that they need not have now).
        // Shallow products (below what gemm_large_kernel takes) run on gemm_tile_kernel in every shape, those of many rows with
        // 256 x 128 tiles where these make no more than a round, else with 256 x 256: 16384 x 512, K 128 9.5 us with the smaller
        // and 10.9 with the larger, 8192 x 3072, K 64 16.9 and 15.8, 16384 x 3072, K 64 27.5 and 23.2.
        const bool many = M > 1024 && dtype == DT_BF16, shallow = K < LARGE_MIN_K;
        const bool model = !shallow && (many || ((mode & GEMM_FEW_ROWS) && M > OP_RATE_ROWS));
        const int max_splits = !many ? 16 : (mode & GEMM_FEW_ROWS) && M <= MAX_SPLIT_ROWS ? 8 : 1;
        const int shallow_cfg = (int64_t)((M + 255) / 256) * ((N + 127) / 128) <= 256 ? C256x128 : C256x256;
        double best = 1e30;
        for (int cfg = 0; cfg < N_CFG; ++cfg) {
            if (CFG[cfg].bm >= 2 * M && CFG[cfg].bm > 64) continue;     // more than half the rows would be padding
            if (cfg == F64x64 || (dtype == DT_F32 && cfg != C64x128)) continue;
            if (only_large(cfg) && !model) continue;
            if ((cfg == C256x160 || (cfg == C256x128 && many && !shallow)) && !(mode & GEMM_FEW_ROWS)) continue;     // a model's launches only
            if (many && (shallow ? cfg != shallow_cfg : !is_large(cfg))) continue;
            for (int s = 1; s <= max_splits; ++s) {
                if (!split_ok(dtype, K, s)) continue;
                if (many && s > 1 && (int64_t)s * M * N * 4 > MANY_ROWS_PARTIALS) break;
                if (s > 1 && 4e-6 + split_cost(s, M, N, mode & GEMM_DEFER, model ? MODEL_RATES : OP_RATES) >= best) break;      // and so would more parts
                double c = plan_cost(dtype, cfg, s, M, N, K, mode & GEMM_DEFER, model && dtype == DT_BF16);
                if (c < best) { best = c; p.cfg = cfg; p.splits = s; }
            }
        }
        p.cost = best;
        if ((mode & GEMM_FEW_ROWS) && M <= (dtype == DT_F32 ? 2048 : 256)) {
            p.stream = gemm_stream_plan(dtype, M, N, K, mode & GEMM_DEFER);
            if (p.stream.nt && (dtype == DT_F32 ? stream_f32_seconds(p.stream, M, N, K) > F32_STREAM_MARGIN * best
                                                : p.stream.cost > STREAM_MARGIN * best)) p.stream = StreamPlan{};
            if (p.stream.nt) p.cost = p.stream.cost;
        }
        if (memo.size() > 4096) memo.clear();
        memo[key] = Choice{p.cfg, p.splits, p.cost, p.stream};
    }
    if (p.stream.nt) {
        p.route = 1;
        p.splits = p.stream.splits;
        return p;
    }
    const Knobs& kn = knobs();
    if (kn.cfg >= 0 && kn.cfg < N_CFG && kn.cfg != F64x64 && dtype == DT_BF16 && !(only_large(kn.cfg) && K < LARGE_MIN_K)) p.cfg = kn.cfg;
    if (kn.split > 0 && split_ok(dtype, K, kn.split)) p.splits = kn.split;
    p.spread = 1;     // never slower than issuing a k-tile's loads at once in that sweep, up to 15 % faster from M = 128 on
    if (kn.spread >= 0) p.spread = kn.spread != 0;
    p.tiles = ((M + CFG[p.cfg].bm - 1) / CFG[p.cfg].bm) * ((N + CFG[p.cfg].bn - 1) / CFG[p.cfg].bn);
    p.k_per_split = split_k_tiles(dtype, K, p.splits) * k_tile(dtype);
    return p;
}

bool gemm_force_ok(int cfg, int splits, int M, int N, int K)
{
    return cfg >= -1 && cfg < N_CFG && cfg != F64x64 && M >= 1 && N % 4 == 0 && K % k_tile(DT_BF16) == 0 && !(only_large(cfg) && K < LARGE_MIN_K) &&
           splits >= 1 && split_ok(DT_BF16, K, splits);
}

// Per-device launch state: the number of persistent workgroups of a tile GEMM (one per compute unit: every bf16
// configuration takes more than half of a CU's LDS, so one workgroup is resident per CU; rounded down to a
// multiple of 8 for the XCD mapping).
static int current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
    return dev;
}
static int persistent_grid()
{
    static std::once_flag once[MAX_DEVICES];
    static int grid[MAX_DEVICES];
    int dev = current_device();
    std::call_once(once[dev], [&]() {
        int cus = 0;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 8) cus = 256;
        grid[dev] = cus / 8 * 8;
        if (knobs().grid >= 8) grid[dev] = knobs().grid / 8 * 8;
    });
    return grid[dev];
}

// A launch of many 256 x 256 tiles runs in rounds of one tile per CU, and a last round that fills few CUs costs as
// much as a full one.  split_rows returns the number of leading rows whose tiles fill whole rounds when handing the
// remaining rows (a few hundred) to a second, separately planned launch is cheaper by the cost model, else M.
static int split_rows(int dtype, int M, int N, int K, int mode)
{
    if (M <= 1024 || dtype != DT_BF16) return M;
    Plan all = make_plan(dtype, M, N, K, mode);
    if (all.route != 0) return M;
    const bool model = (mode & GEMM_FEW_ROWS) && K >= LARGE_MIN_K;          // others are cut by the old rates (see plan_cost)
    int G = persistent_grid();
    int tn = (N + 255) / 256, tm = (M + 255) / 256, total = tm * tn;
    int rounds = total / G;
    if (rounds < 1 || total == rounds * G) return M;
    // Candidates for the first launch: the most row tiles that fill whole rounds, and the largest multiple of 64 row
    // tiles.  With a multiple of 64 every XCD keeps one group of 8 row tiles for the whole launch and all eight walk
    // the weight columns in step; measured, a round of such a launch takes 3-6 % less (16 384 rows against 17 120 -
    // 17 352 at the OPT-13B shape: 1826 us + 127 us for the rest against 2049 us in one launch of 16 rounds).
    int best = M;
    double best_cost = model ? all.cost : plan_cost(dtype, C256x256, 1, M, N, K, false, false);
    int cand[2] = {rounds * G / tn, tm / 64 * 64};
    for (int tm1 : cand) {
        if (tm1 < 1 || tm1 >= tm) continue;
        int M1 = tm1 * 256;
        double first = plan_cost(dtype, C256x256, 1, M1, N, K, false, model);
        if (tm1 % 64 == 0) first *= 0.95;
        double rest = model || M - M1 <= 1024 ? make_plan(dtype, M - M1, N, K, mode & ~GEMM_DEFER).cost
                                              : plan_cost(dtype, C256x256, 1, M - M1, N, K, false, false);
        double parts = first + rest;
        if (parts < best_cost) { best_cost = parts; best = M1; }
    }
    return best;
}

// exe_op_gemm's mode: bf16 by the tile kernel alone
static int op_mode(int dtype) { return dtype == DT_F32 ? GEMM_FEW_ROWS : GEMM_TILE_ONLY; }

// the tile configuration that a plan's launch takes
static int reported_cfg(int dtype, const Plan& p, int M, int N, int K)
{
    if (dtype != DT_F32 || p.route != 0) return p.cfg;
    const int tiles[] = {C128x128, C64x128, F64x64};
    double seconds;
    return tiles[gemm_f32_tile(M, N, K, &seconds)];
}

void gemm_plan_info(int dtype, int M, int N, int K, int* route, int* cfg, int* splits, int* rows_first)
{
    int M1 = split_rows(dtype, M, N, K, op_mode(dtype));
    Plan p = make_plan(dtype, M1, N, K, op_mode(dtype));
    *route = p.route;
    *cfg = reported_cfg(dtype, p, M1, N, K);
    *splits = p.splits;
    *rows_first = M1;
}

size_t gemm_workspace_bytes(int dtype, int M, int N, int K, int mode)
{
    int M1 = split_rows(dtype, M, N, K, mode);
    if (M1 < M) return gemm_workspace_bytes(dtype, M - M1, N, K, mode & ~GEMM_DEFER);
    Plan p = make_plan(dtype, M, N, K, mode);
    return p.splits > 1 ? (size_t)p.splits * M * N * sizeof(float) : 0;
}

template <typename T>
static void reduce_rows(const GemmArgs& a, int splits, int64_t first, int rows, hipStream_t s)
{
    const unsigned quads = (unsigned)((int64_t)rows * (a.N / 4));
    void* out = (char*)a.out + first * a.N * (a.out_mode == OUT_T ? sizeof(T) : sizeof(float));
    splitk_reduce_kernel<T><<<(quads + REDUCE_THREADS - 1) / REDUCE_THREADS, REDUCE_THREADS, 0, s>>>(
        quads, a.N / 4, (int64_t)a.M * a.N, splits, a.workspace + first * a.N, (const T*)a.bias, a.act, a.alpha, a.out_mode, out);
}

hipError_t launch_splitk_reduce(const GemmArgs& a, int splits, hipStream_t s)
{
    const int most = (int)std::min<int64_t>(a.M, REDUCE_QUADS / (a.N / 4));
    for (int64_t first = 0; first < a.M; first += most) {
        const int rows = (int)std::min<int64_t>(most, a.M - first);
        if (a.dtype == DT_F32) reduce_rows<float>(a, splits, first, rows, s);
        else reduce_rows<bf16_t>(a, splits, first, rows, s);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, int BM, int BN, int WM, int WN, int ST>
static hipError_t launch_tile(const GemmArgs& a, const Plan& p, hipStream_t s)
{
    auto kern = gemm_tile_kernel<T, BM, BN, WM, WN, ST>;
    constexpr int threads = (BM / WM) * (BN / WN) * 64;
    constexpr int lds = ST * (BM + BN) * TROW + (threads / 64) * epilogue_cols(BM, BN, WM, WN, ST) * 128;
    static_assert(lds <= 160 * 1024, "LDS budget");
    static LdsLimit limit[MAX_DEVICES];
    hipError_t e = limit[current_device()].raise((const void*)kern, lds);
    if (e != hipSuccess) return e;
    int tm = (a.M + BM - 1) / BM, tn = (a.N + BN - 1) / BN;
    int items = tm * tn * p.splits;
    int gmax = persistent_grid();
    int grid = items < gmax ? items : gmax;
    int w_once = tm == 1 && a.M <= 64;      // measured: 7-10 % faster up to 32 rows, even from 96 rows on
    if (knobs().nt >= 0) w_once = knobs().nt != 0;
    kern<<<grid, threads, lds, s>>>(a.M, a.N, a.K, (const T*)a.A, (const T*)a.W, (const T*)a.bias, a.act, a.alpha, a.out_mode,
                                    a.out, a.workspace, tm, tn, p.k_per_split, p.splits,
                                    (p.spread ? 1 : 0) | (w_once ? 2 : 0), a.lda ? a.lda : a.K, a.ldw ? a.ldw : a.K);
    return hipGetLastError();
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// the generic kernel is the only one that reads and writes float operands element by element
static bool needs_generic(const GemmArgs& a)
{
    return a.dtype == DT_F32 && !(aligned16(a.A) && aligned16(a.W) && aligned16(a.out) && aligned16(a.bias));
}

static int launch_mode(const GemmArgs& a)
{
    return (a.few_rows ? GEMM_FEW_ROWS : 0) | (a.pending && a.out_mode == OUT_RESID && a.alpha == 1.f ? GEMM_DEFER : 0);
}

// Keys and values go straight into the cache from launches of whole sums on the kernels that the rows of an encode batch run on:
// gemm_large_kernel and the float tiles.  Few rows (the streaming kernel, the smaller bf16 tiles, split sums) leave them to a copy
// of their own, 2-4 us.  (In the 256 x 256 shape of gemm_tile_kernel, K < 256, that epilogue would spill 75 registers.)
static bool stores_kv(const GemmArgs& a, int rows, const Plan& p)       // p: the plan of a launch of that many of a's rows
{
    return p.route == 0 && p.splits == 1 && a.out_mode == OUT_T && a.act < 0 && !needs_generic(a) &&
           (a.dtype == DT_F32 || runs_large(p.cfg, rows, a.N, a.K, p.splits));
}

// The launches of a product in the order of their rows, f(first row, rows): one, or where whole rounds of tiles go first (split_rows)
// those rows' own launches and then the others'.  What is launched and what is said about it beforehand both come from here:
// either part may be cut again.
template <typename F> static void each_launch(int dtype, int row, int M, int N, int K, int mode, F&& f)
{
    int M1 = split_rows(dtype, M, N, K, mode);
    if (M1 == M) {
        f(row, M);
        return;
    }
    each_launch(dtype, row, M1, N, K, mode & ~GEMM_DEFER, f);
    each_launch(dtype, row + M1, M - M1, N, K, mode & ~GEMM_DEFER, f);
}

int gemm_kv_rows(const GemmArgs& a)
{
    if (a.M <= 0 || a.force_splits) return 0;
    int stored = 0;
    each_launch(a.dtype, 0, a.M, a.N, a.K, launch_mode(a), [&](int row, int rows) {
        if (stored == row && stores_kv(a, rows, make_plan(a.dtype, rows, a.N, a.K, launch_mode(a)))) stored += rows;
    });
    return stored;
}

int gemm_launches(const GemmArgs& a, int cap, int32_t* rows, int32_t* stores)
{
    int n = 0;
    each_launch(a.dtype, 0, a.M, a.N, a.K, launch_mode(a), [&](int, int M) {
        if (n < cap) {
            rows[n] = M;
            stores[n] = stores_kv(a, M, make_plan(a.dtype, M, a.N, a.K, launch_mode(a)));
        }
        ++n;
    });
    return n;
}

static Plan forced_plan(Plan p, int dtype, int K, int cfg, int splits)
{
    p.route = 0;
    if (cfg >= 0) p.cfg = cfg;
    p.splits = splits;
    p.k_per_split = split_k_tiles(dtype, K, splits) * k_tile(dtype);
    p.spread = 1;
    return p;
}

int gemm_launch_plans(const GemmArgs& a, bool defer, int cap, int32_t* plans)
{
    const int mode = GEMM_FEW_ROWS | (defer ? GEMM_DEFER : 0);
    int n = 0;
    auto put = [&](int rows, const Plan& p) {
        if (n < cap) {
            const int32_t plan[] = {rows, p.route, reported_cfg(a.dtype, p, rows, a.N, a.K), p.splits, 
                                    a.dtype == DT_BF16 && p.route == 0 && runs_large(p.cfg, rows, a.N, a.K, p.splits)};
            std::copy(plan, plan + 5, plans + 5 * n);
        }
        ++n;
    };
    if (a.force_splits) put(a.M, forced_plan(make_plan(a.dtype, a.M, a.N, a.K, mode), a.dtype, a.K, a.force_cfg, a.force_splits));
    else each_launch(a.dtype, 0, a.M, a.N, a.K, mode, [&](int, int rows) {
        put(rows, make_plan(a.dtype, rows, a.N, a.K, rows == a.M ? mode : mode & ~GEMM_DEFER));
    });
    return n;
}

static hipError_t launch_rows(const GemmArgs& a, int mode, hipStream_t s);

hipError_t launch_gemm(const GemmArgs& a, hipStream_t s)
{
    if (a.pending) *a.pending = 0;
    if (a.M <= 0 || a.N <= 0) return hipSuccess;
    const int mode = launch_mode(a);
    if (a.force_splits) {
        GemmArgs plain = a;
        plain.kv = nullptr;
        return launch_rows(plain, mode, s);
    }
    const size_t esz = a.dtype == DT_BF16 ? 2 : 4, osz = a.out_mode == OUT_T ? esz : 4;
    hipError_t e = hipSuccess;
    int stored = 0;                          // leading rows whose keys and values are in the cache: see gemm_kv_rows
    each_launch(a.dtype, 0, a.M, a.N, a.K, mode, [&](int row, int rows) {
        if (e != hipSuccess) return;
        GemmArgs part = a;
        const bool whole = rows == a.M;
        if (!whole) part.pending = nullptr;
        part.M = rows;
        part.A = (const char*)a.A + (size_t)row * (a.lda ? a.lda : a.K) * esz;
        part.out = (char*)a.out + (size_t)row * a.N * osz;
        KvStore kv;
        part.kv = nullptr;
        if (a.kv && stored == row && stores_kv(a, rows, make_plan(a.dtype, rows, a.N, a.K, mode))) {
            kv = *a.kv;
            kv.row += row;
            kv.cap += row;
            part.kv = &kv;
            stored += rows;
        }
        e = launch_rows(part, whole ? mode : mode & ~GEMM_DEFER, s);
    });
    return e;
}

// one launch (and, of split sums, their reduction)
static hipError_t launch_rows(const GemmArgs& a, int mode, hipStream_t s)
{
    Plan p = make_plan(a.dtype, a.M, a.N, a.K, mode);
    if (a.force_splits) p = forced_plan(p, a.dtype, a.K, a.force_cfg, a.force_splits);
    if (needs_generic(a)) p.route = 2;
    if (p.route == 2) {
        dim3 grid((a.N + 63) / 64, (a.M + 63) / 64);
        if (a.dtype == DT_F32)
            gemm_generic_kernel<float><<<grid, 256, 0, s>>>(a.M, a.N, a.K, (const float*)a.A, (const float*)a.W,
                                                            (const float*)a.bias, a.act, a.alpha, a.out_mode, a.out);
        else
            gemm_generic_kernel<bf16_t><<<grid, 256, 0, s>>>(a.M, a.N, a.K, (const bf16_t*)a.A, (const bf16_t*)a.W,
                                                             (const bf16_t*)a.bias, a.act, a.alpha, a.out_mode, a.out);
        return hipGetLastError();
    }
    if (p.splits > 1 && (size_t)p.splits * a.M * a.N * sizeof(float) > (a.workspace ? a.workspace_bytes : 0)) {
        // fewer parts than planned, as the workspace allows (a model's is sized from every eighth row count)
        if (p.route == 1) {
            p.stream = gemm_stream_candidate(a.dtype, p.stream.nt, p.stream.ma, 1, a.M, a.N, a.K, false);
            p.splits = 1;
        } else {
            size_t fit = a.workspace ? a.workspace_bytes / ((size_t)a.M * a.N * sizeof(float)) : 0;
            while (p.splits > 1 && ((size_t)p.splits > fit || !split_ok(a.dtype, a.K, p.splits))) --p.splits;
            p.k_per_split = split_k_tiles(a.dtype, a.K, p.splits) * k_tile(a.dtype);
        }
    }
    hipError_t e;
    if (p.route == 1) e = launch_gemm_stream(a, p.stream, s);
    else if (a.dtype == DT_F32) {
        e = launch_gemm_f32(a, s);
    } else {
        switch (p.cfg) {
            case C64x256: e = launch_tile<bf16_t, 64, 256, 32, 64, 3>(a, p, s); break;
            case C128x256: case C256x256: case C256x128: case C192x256: case C256x160:
                if (runs_large(p.cfg, a.M, a.N, a.K, p.splits)) e = launch_gemm_large(a, CFG[p.cfg].bm, CFG[p.cfg].bn, p.k_per_split, p.splits, persistent_grid(), s);
                else if (p.cfg == C128x256) e = launch_tile<bf16_t, 128, 256, 64, 64, 3>(a, p, s);
                else if (p.cfg == C256x128) e = launch_tile<bf16_t, 256, 128, 64, 64, 3>(a, p, s);
                else e = launch_tile<bf16_t, 256, 256, 128, 64, 2>(a, p, s);
                break;
            case C64x128: e = launch_tile<bf16_t, 64, 128, 32, 64, 4>(a, p, s); break;
            default: e = launch_tile<bf16_t, 128, 128, 64, 64, 3>(a, p, s);
        }
    }
    if (e != hipSuccess || p.splits == 1) return e;
    if (mode & GEMM_DEFER) {
        *a.pending = p.splits;
        return hipSuccess;
    }
    return launch_splitk_reduce(a, p.splits, s);
}

}  // namespace exe
