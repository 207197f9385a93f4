// GEMM for few rows (decode iterations, small batches): every weight is used once or a few times, so the kernel is a
// stream of the weight matrix with some matrix arithmetic behind it.
//
// What bounds it: HBM for large weights, the latency of one load - multiply - reduce chain for small ones.  The tile
// kernel (kernels_gemm.hip) needs split-K over workgroups to fill the chip at these row counts, so each of its launches
// is followed by a reduction kernel (4.5 us), and its waves meet at a barrier per 64 k.  Here a workgroup owns NT * 16
// output features of MA * 8 rows and its waves split K instead: each wave streams its own part of the rows through a
// private LDS ring (direct global->LDS loads, whole 128-byte lines, no barrier in the loop), and the waves' accumulators
// meet once, in LDS, in wave order.  Loading the operands straight into registers was measured first: the MFMA operand
// layout puts neighbouring lanes on different rows, 16 bytes each, which the address unit serves at a quarter of its
// rate (15360 x 5120 weights: 36 us; through LDS 24 us = 6.5 TB/s).
//
// Measured on one MI355X, weights from HBM, tile kernel + reduction -> this kernel, us per launch:
//   bf16 15360 x  5120   1 row 29.5 -> 24.3   16 rows 30.6 -> 25.8   32 rows 32.5 -> 28.9   64 rows 35.5 -> 34.4
//   bf16 20480 x  5120   1 row 37.9 -> 31.3   16 rows 38.6 -> 33.2   32 rows 40.6 -> 35.3   64 rows 45.0 -> 41.6
//   bf16  5120 x  5120   1 row 17.7 -> 11.9   16 rows 16.2 -> 13.6   32 rows 17.2 -> 16.1   64 rows 19.9 -> 22.1
//   bf16  3072 x  1024   1 row  8.5 ->  3.4   48 rows  9.9 ->  5.1   (a 1024-wide model)
//   float  768 x   256   4 rows 35.2 -> 2.6, 400 rows 39.2 -> 4.4 (from the plain-FMA kernel);  256 x 1024  4 rows 134 -> 4.0
#include "gemm_epilogue.h"
#include "kernels.h"

namespace exe {

// Launch shape of an instantiation.  8 waves where a workgroup has only 16 features and at most 16 rows (little to load
// per unit of K, and the waves' sums are cheap to add), else 4.  Stages: as many as leave room for two workgroups on a CU
// (they overlap one's start and end with the other's stream), at least 2, at most 4; more in flight gained nothing.
constexpr int stream_waves(int NT, int MA) { return NT == 1 && MA <= 2 ? 8 : 4; }
constexpr int stream_stages(int NT, int MA)
{
    int kb = stream_waves(NT, MA) * (NT * 2 + MA), st = 80 / kb;
    return st < 2 ? 2 : st > 4 ? 4 : st;
}
constexpr int stream_lds(int NT, int MA)
{
    int ring = stream_waves(NT, MA) * stream_stages(NT, MA) * (NT * 2 + MA) * 1024;
    int red = stream_waves(NT, MA) * NT * ((MA + 1) / 2) * 1024;
    return ring > red ? ring : red;
}

// Rows of a stage: NT * 16 weight rows, then MA * 8 activation rows, 128 bytes each; 16-byte chunk c of row r lies at slot
// c ^ ((r >> 1) & 7), which keeps the fragment reads free of bank conflicts (applied on the global side: lane l of a
// direct-to-LDS load lands at byte 16 * l).
__device__ __forceinline__ int stream_swz(int row) { return (row >> 1) & 7; }

// A norm in front of the product (NORM): the activation rows are norm(x), computed by every workgroup for itself into LDS
// while its first weights arrive, instead of by a launch of its own.  Same layout as in a stage, [unit][row][128 bytes].
template <typename T> struct NormIn {
    const float* x;                  // [.., K]
    const int32_t* row_index;        // nullable
    const T *gain, *shift;           // shift: LayerNorm only
    float eps, out_scale;
    int rms;
    const float* partial;            // [n_part][partial_rows][K], added to x first, and their bias (nullable)
    const T* part_bias;
    int n_part, partial_rows;
    TopLogit* top;                   // nullable
};
constexpr int NORM_STAGES = 3;
// Where it is taken: each workgroup repeats the norm, so the rows have to be few and short.  A launch less (2.4 us on the GPU, 2.6
// to enqueue) against its norm: decode iterations of a 256-wide float model 1.15x, of a 512-wide encoder-decoder 1.12x;
// 1024 wide with 4 to 16 rows 0.98-0.99x.
constexpr int NORM_MAX_K = 512, NORM_MAX_ROWS = 16, NORM_MAX_N = 4096;
// With partial sums to add first (a small model's last feed-forward block in front of the LM head), each workgroup reads all of them:
// 512 KB (8 rows of 256 in 64 parts, 4 of 512) 67 and 79 us a decode iteration against 75 and 87 with a norm of its own, 1 MB 87
// and 90, 2 MB 106 and 100.
constexpr int64_t NORM_MAX_PART_BYTES = 1 << 20;
constexpr int NORM_Q = NORM_MAX_K / 256;     // groups of 4 elements per lane and row
template <typename T> constexpr int norm_lds(int MA, int K) { return stream_waves(1, MA) * NORM_STAGES * 2048 + MA * 8 * K * (int)sizeof(T); }

// rows w, w + NW, .. of the workgroup's M by wave w; K % 32 == 0
template <typename T, int NW, int MA>
__device__ __forceinline__ void norm_rows(const NormIn<T>& in, int M, int K, int wave, int lane, unsigned char* dst, const f32x4 (&g)[NORM_Q],
                                          const f32x4 (&b)[NORM_Q], const f32x4 (&v)[2][NORM_Q])
{
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int r = wave + i * NW;
        if (r >= M || r >= MA * 8) continue;
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < NORM_Q; ++q)
#pragma unroll
            for (int j = 0; j < 4; ++j) s += in.rms ? v[i][q][j] * v[i][q][j] : v[i][q][j];
        float tot = wave_sum(s), mean = 0.f, var = tot / K;
        if (!in.rms) {
            mean = tot / K;
            float sq = 0.f;
#pragma unroll
            for (int q = 0; q < NORM_Q; ++q)
                if ((q * 64 + lane) * 4 < K)
#pragma unroll
                    for (int j = 0; j < 4; ++j) sq += (v[i][q][j] - mean) * (v[i][q][j] - mean);
            var = wave_sum(sq) / K;
        }
        float rstd = 1.f / sqrtf(var + in.eps);
#pragma unroll
        for (int q = 0; q < NORM_Q; ++q) {
            int k = (q * 64 + lane) * 4, byte = k * (int)sizeof(T);
            if (k >= K) continue;
            typename Vec4<T>::type y;
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = (T)(((v[i][q][j] - mean) * rstd * g[q][j] + b[q][j]) * in.out_scale);
            *(typename Vec4<T>::type*)(dst + (byte / 128 * (MA * 8) + r) * 128 + ((((byte & 127) >> 4) ^ stream_swz(r)) << 4) + (byte & 15)) = y;
        }
    }
}

// A "unit" of K is 128 bytes of a row.  Workgroup z of a split takes units z * units_per_split ..; wave w of it the units
// w, w + waves, ... of those, so that at any time the workgroup reads neighbouring lines of its rows.  n_split > 1:
// float partials [split][M][N], summed by the split-K reduction.
template <typename T, int NT, int MA, bool NORM>
__device__ __forceinline__ void stream_body(
    int M, int N, int K, const T* __restrict__ A, const T* __restrict__ W, const T* __restrict__ bias, int act, float alpha,
    int out_mode, void* __restrict__ out, float* __restrict__ partial, int units_per_split, int n_split, int lda, int ldw,
    const NormIn<T>& norm)
{
    constexpr int NW = stream_waves(NT, MA), ST = NORM ? NORM_STAGES : stream_stages(NT, MA);
    constexpr int MT = (MA + 1) / 2;                 // 16-row MFMA tiles (8 rows: the upper half repeats the lower one)
    constexpr int L = NT * 2 + (NORM ? 0 : MA);      // 1 KB loads per unit: 8 rows each
    constexpr int STAGE = L * 1024;
    static_assert(L * (ST - 1) <= 63, "vmcnt range");
    extern __shared__ __align__(16) unsigned char lds[];
    int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int fr = lane & 15, g = lane >> 4;
    int n0 = blockIdx.x * NT * 16, m0 = blockIdx.y * MA * 8, z = blockIdx.z;
    int u = z * units_per_split, u_end = K / (128 / (int)sizeof(T));
    if (u + units_per_split < u_end) u_end = u + units_per_split;
    u += wave;
    int nu = u < u_end ? (u_end - u + NW - 1) / NW : 0;

    // rows past the edge repeat the last row; their results are not stored
    int wrows = N - n0 < NT * 16 ? N - n0 : NT * 16, arows = M - m0 < MA * 8 ? M - m0 : MA * 8;
    const char* src_w = (const char*)(W + (int64_t)n0 * ldw) + (int64_t)u * 128;
    const char* src_a = NORM ? nullptr : (const char*)(A + (int64_t)m0 * lda) + (int64_t)u * 128;
    unsigned off_w[NT * 2], off_a[MA];
#pragma unroll
    for (int p = 0; p < NT * 2; ++p) {
        int r = p * 8 + (lane >> 3);
        off_w[p] = (unsigned)(r < wrows ? r : wrows - 1) * (unsigned)(ldw * (int)sizeof(T)) + (((lane & 7) ^ stream_swz(r)) << 4);
    }
#pragma unroll
    for (int p = 0; p < MA; ++p) {
        int r = p * 8 + (lane >> 3);
        off_a[p] = (unsigned)(r < arows ? r : arows - 1) * (unsigned)(lda * (int)sizeof(T)) + (((lane & 7) ^ stream_swz(r)) << 4);
    }
    const unsigned char* ring = lds + wave * (ST * STAGE);
    unsigned ring_at = (unsigned)(size_t)(__attribute__((address_space(3))) const unsigned char*)ring;
    const bool w_once = gridDim.y == 1;              // read once: nontemporal, so that it does not displace A in L2
    // inline assembly: the compiler would put a vmcnt(0) in front of every LDS read behind a direct-to-LDS load it knows of
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    auto load_to_lds = [&](const char* src, unsigned voff, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
    auto load_to_lds_nt = [&](const char* src, unsigned voff, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
#pragma clang diagnostic pop
    auto issue = [&](int i, int st) {
        unsigned dst = ring_at + st * STAGE;
        const char* w = src_w + (int64_t)i * (NW * 128);
        const char* a = src_a + (int64_t)i * (NW * 128);
#pragma unroll
        for (int p = 0; p < NT * 2; ++p) {
            if (w_once) load_to_lds_nt(w, off_w[p], dst + p * 1024);
            else load_to_lds(w, off_w[p], dst + p * 1024);
        }
        if constexpr (!NORM) {
#pragma unroll
            for (int p = 0; p < MA; ++p) load_to_lds(a, off_a[p], dst + (NT * 2 + p) * 1024);
        }
    };
    unsigned char* normed = lds + NW * ST * STAGE;   // NORM: all K of the activation rows
    // weight rows feed the MFMA's A operand, activation rows its B operand: a lane's accumulator is then 4 consecutive
    // output features 4 * g .. of one row fr
    f32x4 acc[NT][MT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < MT; ++j) acc[t][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto consume = [&](int st, int i) {
        const unsigned char* s = ring + st * STAGE;
        const unsigned char* sa = NORM ? normed + (u + i * NW) * (MA * 1024) : s + NT * 2048;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            u32x4 fw[NT], fa[MT];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                int r = t * 16 + fr;
                fw[t] = *(const u32x4*)(s + r * 128 + (((h * 4 + g) ^ stream_swz(r)) << 4));
            }
#pragma unroll
            for (int j = 0; j < MT; ++j) {
                int r = MA == 1 ? (fr & 7) : j * 16 + fr;
                fa[j] = *(const u32x4*)(sa + r * 128 + (((h * 4 + g) ^ stream_swz(r)) << 4));
            }
#pragma unroll
            for (int t = 0; t < NT; ++t)
#pragma unroll
                for (int j = 0; j < MT; ++j) acc[t][j] = HalfUnit<T>::mma(fw[t], fa[j], acc[t][j]);
        }
    };
    // The ring is the wave's own: its vmcnt says when a stage has landed, its lgkmcnt when the reads of the stage that is
    // filled again are done.
    f32x4 ng[NORM_Q], nb[NORM_Q], nv[2][NORM_Q];
    if constexpr (NORM) {                            // the norm's operands go out ahead of the first weights
        const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < NORM_Q; ++q) {
            int k = (q * 64 + lane) * 4;
            ng[q] = nb[q] = nv[0][q] = nv[1][q] = zero;
            if (k >= K) continue;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                int r = wave + i * NW;
                if (r >= M) continue;
                int64_t at = (int64_t)(norm.row_index ? norm.row_index[r] : r) * K + k;
                nv[i][q] = *(const f32x4*)(norm.x + at);
                if (!norm.n_part) continue;
                f32x4 sum = zero;
                const float* p = norm.partial + at;
                int64_t slice = (int64_t)norm.partial_rows * K;
                int s = 0;
                for (; s + 16 <= norm.n_part; s += 16) {
                    f32x4 pv[16];
#pragma unroll
                    for (int j = 0; j < 16; ++j) pv[j] = *(const f32x4*)(p + (s + j) * slice);
#pragma unroll
                    for (int j = 0; j < 16; ++j) sum += pv[j];
                }
                for (; s + 4 <= norm.n_part; s += 4) {
                    f32x4 p0 = *(const f32x4*)(p + s * slice), p1 = *(const f32x4*)(p + (s + 1) * slice);
                    f32x4 p2 = *(const f32x4*)(p + (s + 2) * slice), p3 = *(const f32x4*)(p + (s + 3) * slice);
                    sum += p0; sum += p1; sum += p2; sum += p3;
                }
                for (; s < norm.n_part; ++s) sum += *(const f32x4*)(p + s * slice);
                if (norm.part_bias) {
                    typename Vec4<T>::type pb = *(const typename Vec4<T>::type*)(norm.part_bias + k);
#pragma unroll
                    for (int j = 0; j < 4; ++j) sum[j] += (float)pb[j];
                }
                nv[i][q] += sum;
            }
            typename Vec4<T>::type gt = *(const typename Vec4<T>::type*)(norm.gain + k);
#pragma unroll
            for (int j = 0; j < 4; ++j) ng[q][j] = (float)gt[j];
            if (!norm.rms) {
                typename Vec4<T>::type bt = *(const typename Vec4<T>::type*)(norm.shift + k);
#pragma unroll
                for (int j = 0; j < 4; ++j) nb[q][j] = (float)bt[j];
            }
        }
    }
#pragma unroll
    for (int d = 0; d < ST - 1; ++d)
        if (d < nu) issue(d, d);
    if constexpr (NORM) {
        norm_rows<T, NW, MA>(norm, M, K, wave, lane, normed, ng, nb, nv);
        __syncthreads();
    }
    int st = 0, fill = ST - 1, i = 0;
    for (; i + ST - 1 < nu; ++i) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue(i + ST - 1, fill);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(L * (ST - 1)) : "memory");
        consume(st, i);
        fill = st;
        st = st + 1 == ST ? 0 : st + 1;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    for (; i < nu; ++i) {
        consume(st, i);
        st = st + 1 == ST ? 0 : st + 1;
    }
    __syncthreads();                                 // every wave has read its last stage: the rings become the sum buffer
    f32x4* red = (f32x4*)lds;                        // [wave][tile][lane]
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int j = 0; j < MT; ++j) red[(wave * NT * MT + t * MT + j) * 64 + lane] = acc[t][j];
    __syncthreads();
    for (int x = wave; x < NT * MT; x += NW) {
        f32x4 v = red[x * 64 + lane];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += red[(w * NT * MT + x) * 64 + lane];
        int m = m0 + (x % MT) * 16 + fr, n = n0 + (x / MT) * 16 + 4 * g;
        if (NORM && norm.top) {                      // uniform
            float best = -INFINITY;
            int idx = 0x7fffffff;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (n + j < N) argmax_take(best, idx, v[j], n + j);
            argmax_column(best, idx);
            if (g == 0 && m < M) norm.top[blockIdx.x * 16 + fr] = TopLogit{best, idx};
        }
        if (m >= M || n >= N || (MA == 1 && fr >= 8)) continue;
        if (n_split > 1) *(f32x4*)(partial + ((int64_t)z * M + m) * N + n) = v;
        else epilogue_store4<T>(v, m, n, N, bias, act, alpha, out_mode, out);
    }
}

template <typename T, int NT, int MA>
__global__ __launch_bounds__(stream_waves(NT, MA) * 64) void gemm_stream_kernel(
    int M, int N, int K, const T* __restrict__ A, const T* __restrict__ W, const T* __restrict__ bias, int act, float alpha,
    int out_mode, void* __restrict__ out, float* __restrict__ partial, int units_per_split, int n_split, int lda, int ldw)
{
    stream_body<T, NT, MA, false>(M, N, K, A, W, bias, act, alpha, out_mode, out, partial, units_per_split, n_split, lda, ldw, NormIn<T>{});
}

template <typename T, int MA>
__global__ __launch_bounds__(stream_waves(1, MA) * 64) void norm_stream_kernel(
    int M, int N, int K, const T* __restrict__ W, const T* __restrict__ bias, int act, float alpha, int out_mode,
    void* __restrict__ out, NormIn<T> norm)
{
    stream_body<T, 1, MA, true>(M, N, K, nullptr, W, bias, act, alpha, out_mode, out, nullptr, K / (128 / (int)sizeof(T)), 1, K, K, norm);
}

// ---------------------------------------------------------------- host side
static const int STREAM_NT[] = {1, 2, 4, 5}, STREAM_MA[] = {1, 2, 4, 6, 8};

// Seconds of a launch with these parameters.  Two rates, fitted to the launches named at the top of this file and to 6
// row counts x 16 weight shapes around them (within 10 % of the measured time for most, 20 % at worst): the weights come
// from memory at 6.9 TB/s, and a CU takes in the rows of its workgroups, activations included, at 50 GB/s; the two overlap
// for the most part (third-power mean).  Partial sums cost their round trip, and a reduction launch unless the next kernel takes them (`defer`).  Float adds the MFMA rate of a CU (0.55 TFLOP/s).  2.5 us are paid by every launch.
static double stream_cost(int dtype, int nt, int ma, int splits, int M, int N, int K, bool defer)
{
    double e = dtype == DT_F32 ? 4.0 : 2.0;
    double wgs = (double)((N + nt * 16 - 1) / (nt * 16)) * ((M + ma * 8 - 1) / (ma * 8)) * splits;
    double rounds = (double)(int64_t)((wgs + 255) / 256);
    double per = (double)K / splits;
    double a = (double)N * K * e / 6.9e12;
    double b = rounds * (nt * 16 + ma * 8) * per * e / 50e9;
    double c = dtype == DT_F32 ? rounds * 2.0 * nt * 16 * ((ma + 1) / 2 * 16) * per / 0.55e12 : 0.0;
    double t = 2.5e-6 + cbrt(a * a * a + b * b * b + c * c * c);
    if (stream_waves(nt, ma) * 2 * (nt * 2 + ma) > 80) t += (rounds - 1) * 2e-6;       // one workgroup per CU: rounds do not overlap
    if (splits > 1) t += defer ? 0.5e-6 + 2.0 * splits * M * N * 4 / 8e12 : 3.5e-6 + 2.0 * splits * M * N * 4 / 4e12;
    return t;
}

// Seconds of a float launch, where it is compared with the float tiles: stream_cost, which ranks the candidates, is 14 % low there.
// Fitted to the launches of up to 2048 rows (see F32_STREAM_MARGIN) that take more than 11.5 us: within 4.4 % on average, 13 % at worst.
double stream_f32_seconds(const StreamPlan& p, int M, int N, int K)
{
    double wgs = (double)((N + p.nt * 16 - 1) / (p.nt * 16)) * ((M + p.ma * 8 - 1) / (p.ma * 8));
    double rounds = (double)(int64_t)((wgs + 255) / 256);
    double t = 3.9e-6 + rounds * (0.63e-6 + 2.0 * p.nt * 16 * ((p.ma + 1) / 2 * 16) * K / 0.427e12), w = (double)N * K * 4 / 6.9e12;
    return t > w ? t : w;
}

// the parameters of one candidate; nt = 0 if the shape does not allow it.  Float is not split over workgroups (no workspace
// is asked of its callers); a bf16 part keeps at least 16 units, 4 for each wave.
StreamPlan gemm_stream_candidate(int dtype, int nt, int ma, int splits, int M, int N, int K, bool defer)
{
    int ue = dtype == DT_F32 ? 32 : 64, units = K / ue, per = splits < 1 ? 0 : (units + splits - 1) / splits;
    if (M < 1 || N % 4 != 0 || K % ue != 0 || splits < 1) return StreamPlan{};
    if ((int64_t)K * (dtype == DT_F32 ? 4 : 2) * (nt * 16 > ma * 8 ? nt * 16 : ma * 8) >= ((int64_t)1 << 32)) return StreamPlan{};    // row offsets are 32 bits
    if (splits > 1 && (dtype == DT_F32 || per < 16 || per * (splits - 1) >= units)) return StreamPlan{};
    return StreamPlan{nt, ma, splits, per, stream_cost(dtype, nt, ma, splits, M, N, K, defer)};
}

StreamPlan gemm_stream_plan(int dtype, int M, int N, int K, bool defer)
{
    StreamPlan best;
    for (int nt : STREAM_NT)
        for (int ma : STREAM_MA) {
            if (ma > 1 && (ma - 1) * 8 >= M + 7) continue;            // rows that do not exist
            for (int s = 1; s <= 8; s *= 2) {
                StreamPlan p = gemm_stream_candidate(dtype, nt, ma, s, M, N, K, defer);
                if (!p.nt) break;
                if (!best.nt || p.cost < best.cost) best = p;
            }
        }
    return best;
}

template <typename T, int NT, int MA>
static hipError_t launch_stream(const GemmArgs& a, const StreamPlan& p, hipStream_t s)
{
    auto kern = gemm_stream_kernel<T, NT, MA>;
    constexpr int lds = stream_lds(NT, MA);
    static_assert(lds <= 160 * 1024, "LDS budget");
    static LdsLimit limit[MAX_DEVICES];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
    hipError_t e = limit[dev].raise((const void*)kern, lds);
    if (e != hipSuccess) return e;
    dim3 grid((a.N + NT * 16 - 1) / (NT * 16), (a.M + MA * 8 - 1) / (MA * 8), p.splits);
    kern<<<grid, stream_waves(NT, MA) * 64, lds, s>>>(a.M, a.N, a.K, (const T*)a.A, (const T*)a.W, (const T*)a.bias, a.act, a.alpha,
                                                      a.out_mode, a.out, a.workspace, p.units_per_split, p.splits,
                                                      a.lda ? a.lda : a.K, a.ldw ? a.ldw : a.K);
    return hipGetLastError();
}

template <typename T, int MA> static hipError_t launch_norm_stream(const NormArgs& n, const GemmArgs& a, hipStream_t s)
{
    auto kern = norm_stream_kernel<T, MA>;
    static_assert(norm_lds<T>(MA, NORM_MAX_K) <= 160 * 1024, "LDS budget");
    static LdsLimit limit[MAX_DEVICES];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
    hipError_t e = limit[dev].raise((const void*)kern, norm_lds<T>(MA, NORM_MAX_K));
    if (e != hipSuccess) return e;
    NormIn<T> in{n.x, n.row_index, (const T*)n.gain, (const T*)n.shift, n.eps, n.out_scale, n.rms, n.partial, (const T*)n.bias, n.partial ? n.splits : 0, n.partial_rows, n.top};
    kern<<<dim3((a.N + 15) / 16), stream_waves(1, MA) * 64, norm_lds<T>(MA, a.K), s>>>(
        a.M, a.N, a.K, (const T*)a.W, (const T*)a.bias, a.act, a.alpha, a.out_mode, a.out, in);
    return hipGetLastError();
}

bool norm_gemm_fits(const NormArgs& n, const GemmArgs& a)
{
    uintptr_t any = (uintptr_t)n.x | (uintptr_t)n.gain | (uintptr_t)n.shift | (uintptr_t)a.W | (uintptr_t)a.out | (uintptr_t)a.bias | (uintptr_t)n.partial | (uintptr_t)n.bias;
    return a.M >= 1 && a.M <= NORM_MAX_ROWS && a.K <= NORM_MAX_K && a.K % (a.dtype == DT_F32 ? 32 : 64) == 0 && a.N % 4 == 0 &&
           a.N <= NORM_MAX_N && a.out_mode != OUT_RESID && (!n.partial || (n.last && (int64_t)n.splits * a.M * a.K * 4 <= NORM_MAX_PART_BYTES)) && n.rows == a.M && n.d == a.K && (any & 15) == 0;
}

hipError_t launch_norm_gemm(const NormArgs& n, const GemmArgs& a, hipStream_t s)
{
    if (a.dtype == DT_F32) return a.M <= 8 ? launch_norm_stream<float, 1>(n, a, s) : launch_norm_stream<float, 2>(n, a, s);
    return a.M <= 8 ? launch_norm_stream<bf16_t, 1>(n, a, s) : launch_norm_stream<bf16_t, 2>(n, a, s);
}

hipError_t launch_gemm_stream(const GemmArgs& a, const StreamPlan& p, hipStream_t s)
{
#define EXE_STREAM_MA(T, NT)                                                     \
    switch (p.ma) {                                                              \
        case 1: return launch_stream<T, NT, 1>(a, p, s);                         \
        case 2: return launch_stream<T, NT, 2>(a, p, s);                         \
        case 4: return launch_stream<T, NT, 4>(a, p, s);                         \
        case 6: return launch_stream<T, NT, 6>(a, p, s);                         \
        default: return launch_stream<T, NT, 8>(a, p, s);                        \
    }
#define EXE_STREAM(T)                                                            \
    switch (p.nt) {                                                              \
        case 1: EXE_STREAM_MA(T, 1)                                              \
        case 2: EXE_STREAM_MA(T, 2)                                              \
        case 4: EXE_STREAM_MA(T, 4)                                              \
        default: EXE_STREAM_MA(T, 5)                                             \
    }
    if (a.dtype == DT_F32) { EXE_STREAM(float) }
    else { EXE_STREAM(bf16_t) }
#undef EXE_STREAM
#undef EXE_STREAM_MA
}

}  // namespace exe
