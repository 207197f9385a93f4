// What the two tile GEMMs share (kernels_gemm.hip, kernels_gemm_large.hip): the LDS layout of a stage, the counted waits, and
// the epilogue that turns a wave's accumulators through LDS.
#pragma once
#include "gemm_epilogue.h"
#include "kernels.h"

// EXE_GEMM_ABLATE (a compile-time bit mask, 0 in the library proper) builds measurement variants of the two tile kernels
// whose results are meaningless and whose timing isolates a part: bit 0 drops the MFMAs (the fragment reads from
// LDS go with them), bit 1 drops the loads of the activation tiles, bit 2 the loads of the weight tiles, bit 5 the
// epilogue (no output is written; a split-K reduction still runs, on whatever the workspace holds).  What
// remains keeps its waits, barriers, epilogue and split-K reduction.  `python -m paper_2404_07947_amd.build
// --variant ablate1 -DEXE_GEMM_ABLATE=1` builds libexe_ablate1.so beside the library.
#ifndef EXE_GEMM_ABLATE
#define EXE_GEMM_ABLATE 0
#endif

namespace exe {

// LDS tile layout for a stage of 64 bf16 (32 float) along K: row r is 128 bytes = 8 chunks of 16 bytes; chunk c is
// stored at slot c ^ ((r>>1)&7), so that 16 consecutive rows read at the same chunk index touch 16 distinct
// 16-byte bank groups (256 bytes of banks; measured: zero LDS bank conflicts).
constexpr int TROW = 128;                                   // bytes of K per stage
template <typename T> constexpr int tbk() { return TROW / (int)sizeof(T); }
__device__ __forceinline__ int lds_swz(int row) { return (row >> 1) & 7; }
__device__ __forceinline__ int lds_off(int row, int chunk) { return row * 128 + ((chunk ^ lds_swz(row)) << 4); }

typedef __attribute__((address_space(3))) void* lds_ptr_t;
typedef __attribute__((address_space(1))) const void* gbl_ptr_t;

// s_waitcnt vmcnt(N) lgkmcnt(L) with expcnt at its maximum; vmcnt is split over bits [3:0] and [15:14],
// lgkmcnt is bits [11:8]
template <int N, int L> __device__ __forceinline__ void wait_cnt()
{
    __builtin_amdgcn_s_waitcnt(0x0070 | (N & 15) | ((N >> 4) << 14) | (L << 8));
}

// ---------------------------------------------------------------- tile epilogue
// A lane of a 16x16 accumulator tile holds 4 consecutive output features n = 4*(l/16) .. +3 of one row m = l%16:
// stored as it lies, a wave-wide store would scatter 16-byte pieces over 16 output rows.  Each wave therefore
// turns its tiles through a private LDS buffer, a "group" of 32 rows x EN columns (2 x EN/16 tiles) at a time,
// with the 16-byte slots XOR-swizzled by row so that neither side has bank conflicts, and then stores whole
// row segments.
//
// The LDS accesses are written as inline assembly on purpose: the compiler assumes that a DS read may alias the
// destination of the direct global->LDS loads still in flight for the next item and would put a vmcnt(0) in
// front of every one of them, which also waits for the stores of the previous group.  The buffer is private to
// the wave and is never a destination of those loads; DS operations of one wave execute in order, and the
// lgkmcnt(0) after the reads completes them before the next group's writes.
enum EpiMode { EPI_PARTIAL = 0, EPI_F32, EPI_RESID, EPI_T, EPI_T_RELU, EPI_T_GELU, EPI_T_KV };

// EPI_T_KV: a lane's rows of the 32 that a wave stores next, as KvStore gives them.  What it is for: the keys and values of an
// encode batch were written to the projection's output, read by a kernel that copied them into the cache, and written there; now
// they are written once, and prefill attention reads them there.  A copy took 292 us a layer behind 12288 tokens of the T5-11B
// shape's cross-attention and 12 us behind 8192 tokens of a 1024-wide model; whole encode calls: 75.9 -> 72.8 ms (T5-11B, 16
// prompts), 2234 -> 2160 us (16 prompts, six 1024-wide layers), 781 -> 758 us (32 float prompts, two layers), 7546 -> 7406 us (one
// prompt, 20 OPT-13B layers).
template <int P> struct KvRows {
    int64_t row[P];
    int32_t cap[P];
    template <typename F> __device__ __forceinline__ void load(const KvStore& kv, int M, F m_of)
    {
#pragma unroll
        for (int p = 0; p < P; ++p) {
            int m = m_of(p) < M ? m_of(p) : M - 1;
            row[p] = kv.row[m];
            cap[p] = kv.cap[m];
        }
    }
    // element offset of the first of the wave's features `c0` (uniform, >= first_col) in row p
    __device__ __forceinline__ int64_t at(const KvStore& kv, int p, int c0) const
    {
        int c = c0 - kv.first_col;
        return kv_at(row[p], cap[p], kv.head0 + (c >> kv.dh_shift), kv.dh_shift) + (c & ((1 << kv.dh_shift) - 1));
    }
};

template <int QW> struct LdsTurn;
template <> struct LdsTurn<4> {
    static __device__ __forceinline__ void read(f32x4 (&v)[4], const unsigned (&a)[4])
    {
        asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2]), "=&v"(v[3])
                     : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
                     : "memory");
    }
};
template <> struct LdsTurn<3> {
    static __device__ __forceinline__ void read(f32x4 (&v)[3], const unsigned (&a)[3])
    {
        asm volatile("ds_read_b128 %0, %3\n\tds_read_b128 %1, %4\n\tds_read_b128 %2, %5\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1]), "=&v"(v[2])
                     : "v"(a[0]), "v"(a[1]), "v"(a[2])
                     : "memory");
    }
};
template <> struct LdsTurn<2> {
    static __device__ __forceinline__ void read(f32x4 (&v)[2], const unsigned (&a)[2])
    {
        asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %3\n\ts_waitcnt lgkmcnt(0)"
                     : "=&v"(v[0]), "=&v"(v[1])
                     : "v"(a[0]), "v"(a[1])
                     : "memory");
    }
};

// acc[i][j]: the wave's accumulator tiles (i: 16 output features, j: 16 rows); stg: LDS byte address of the wave's
// buffer (EN * 128 bytes); (row0, col0): output coordinates of the wave's first element; fout: float destination
// of EPI_PARTIAL / EPI_F32 / EPI_RESID; tout: bf16 destination of EPI_T*.
template <typename T, int TM, int TN, int EN, int MODE>
__device__ __forceinline__ void epilogue_tiles(const f32x4 (&acc)[TN][TM], unsigned stg, int lane, int row0, int col0,
                                               int M, int N, const T* __restrict__ bias, float alpha,
                                               float* __restrict__ fout, T* __restrict__ tout, const KvStore& kv = KvStore{})
{
    static_assert(TM % 2 == 0 && TN % (EN / 16) == 0, "groups are 2 tiles high");
    constexpr int QW = EN / 8;                  // 16-byte slots a lane writes, and reads, per group
    constexpr int IW = EN / 16;                 // tiles side by side in a group
    constexpr int NG = TN / IW;                 // groups per 32 rows
    constexpr int G = (TM / 2) * NG;
    constexpr int RPP = EN == 32 ? 8 : 16;      // output rows covered by one wave-wide read
    constexpr int D = G < 2 ? G : 2;            // residual prefetch depth in groups (registers: D * QW * 4)
    int lm = lane & 15, lq = lane >> 4;
    int rc = EN == 32 ? (lane & 7) : (lane & 3);
    int rr = EN == 32 ? (lane >> 3) : (lane >> 2);
    // slot of (row m, 16-byte column c) in the buffer
    auto slot = [](int m, int c) { return EN == 32 ? m * 8 + (c ^ ((m >> 1) & 7)) : m * 4 + (c ^ ((m >> 2) & 3)); };
    unsigned waddr[QW], raddr[QW];
#pragma unroll
    for (int x = 0; x < QW; ++x) {
        int jj = x / IW, ii = x % IW;           // tile (ii, jj) of the group
        waddr[x] = stg + slot(jj * 16 + lm, ii * 4 + lq) * 16;
        raddr[x] = stg + slot(x * RPP + rr, rc) * 16;
    }
    // group g = jp * NG + ig covers rows row0 + 32 jp .. +31 and columns col0 + EN ig .. + EN - 1
    auto g_row = [&](int g, int p) { return row0 + (g / NG) * 32 + p * RPP + rr; };
    auto g_col = [&](int g) { return col0 + (g % NG) * EN + rc * 4; };
    f32x4 bv[NG];
    if (MODE != EPI_PARTIAL) {
#pragma unroll
        for (int x = 0; x < NG; ++x) {
            int n = g_col(x);
            bv[x] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (bias && n < N) {
                typename Vec4<T>::type b = *(const typename Vec4<T>::type*)(bias + n);
#pragma unroll
                for (int e = 0; e < 4; ++e) bv[x][e] = (float)b[e];
            }
        }
    }
    KvRows<QW> kr;
    f32x4 res[D][QW];
    auto load_res = [&](int g) {
        int n = g_col(g);
#pragma unroll
        for (int p = 0; p < QW; ++p) {
            int m = g_row(g, p);
            res[g % D][p] = (m < M && n < N) ? *(const f32x4*)(fout + (int64_t)m * N + n) : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    };
    if (MODE == EPI_RESID) {
#pragma unroll
        for (int g = 0; g < D; ++g) load_res(g);
    }
#pragma unroll
    for (int g = 0; g < G; ++g) {
        int jp = g / NG, ig = g % NG;
        if (MODE == EPI_T_KV && ig == 0) kr.load(kv, M, [&](int p) { return g_row(g, p); });
#pragma unroll
        for (int x = 0; x < QW; ++x) {
            f32x4 vv = acc[ig * IW + x % IW][jp * 2 + x / IW];
            asm volatile("ds_write_b128 %0, %1" ::"v"(waddr[x]), "v"(vv) : "memory");
        }
        f32x4 v[QW];
        LdsTurn<QW>::read(v, raddr);
        int n = g_col(g);
#pragma unroll
        for (int p = 0; p < QW; ++p) {
            int m = g_row(g, p);
            if (m >= M || n >= N) continue;
            int64_t o = (int64_t)m * N + n;
            if (MODE == EPI_PARTIAL) {
                *(f32x4*)(fout + o) = v[p];
            } else {
                f32x4 r = v[p] * alpha + bv[ig];
                if (MODE == EPI_F32) *(f32x4*)(fout + o) = r;
                else if (MODE == EPI_RESID) *(f32x4*)(fout + o) = res[g % D][p] + r;
                else {
                    typename Vec4<T>::type w;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        w[e] = (T)(MODE == EPI_T_RELU ? act_apply(r[e], 0) : MODE == EPI_T_GELU ? act_apply(r[e], 1) : r[e]);
                    T* dst = tout + o;
                    if (MODE == EPI_T_KV && col0 + EN * ig >= kv.first_col) dst = (T*)kv.pool + kr.at(kv, p, col0 + EN * ig) + rc * 4;
                    *(typename Vec4<T>::type*)dst = w;
                }
            }
        }
        if (MODE == EPI_RESID && g + D < G) load_res(g + D);
        __builtin_amdgcn_sched_barrier(0);      // keeps the groups in order: hoisted loads would cost registers
    }
}

}  // namespace exe
