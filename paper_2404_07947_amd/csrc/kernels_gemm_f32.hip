// GEMM in float for many rows, on the bf16 matrix pipes.
//
// What bounds a float product: 16x16x4 float MFMAs, a sixteenth of the bf16 rate.  A float is the sum of three bf16 values without a
// bit lost (h = x rounded, m = x - h rounded, l = x - h - m, 8 bits each), and a product of two floats their nine products, of
// which the three smallest are left out (m l and l m, below 2^-25 of the product each and of either sign, and l l, below 2^-34; all
// three together below 2^-24): six bf16 MFMAs of 32 k in the place of eight float ones of 4, at 16 times the rate.  Sums stay float,
// with fewer roundings on the way: error against 64 bits: see the table at gemm_f32_tile.  Where what is left out adds up with one sign, the
// roundings outweigh it: rows of one random constant times features of another, rms (largest) error of the float MFMAs 2.3e-7 (5.1e-7)
// at K 32, 1.9e-6 (3.8e-6) at 256, 1.5e-5 (3.1e-5) at 2048; here 2.8e-8 (1.1e-7), 6.0e-7 (2.8e-6), 4.1e-6 (2.0e-5), and the same with
// m l and l m taken too, from K 64 on to all three digits, for 10 % more time.
//
// A workgroup of 4 waves splits each operand tile once, on its way from registers to LDS (per wave and fragment it would be as much
// vector work as the MFMAs take); two to four workgroups on a CU, so that one's splitting runs beside another's MFMAs.
//
// What is split is the element times 2^24 (PART_SCALE), so that the parts of small ones stay in bf16's range.  An infinite or NaN
// element, one of 2^104 and more, or a sum of 2^80 and more does not stay in it: tiles with sums that are not finite are computed
// again with float MFMAs (rare, so not for speed).
#include <type_traits>

#include "gemm_tile.h"
#include "kernels.h"

namespace exe {

constexpr int F32_BK = 32, F32_THREADS = 256;
constexpr int F32_ROW = F32_BK * 2;                          // bytes of a row of one plane
constexpr int f32_lds(int BM, int BN) { return 3 * (BM + BN) * F32_ROW > 4 * 4096 ? 3 * (BM + BN) * F32_ROW : 4 * 4096; }

// A plane holds [rows][32 bf16]; 16-byte chunk c of row r at slot c ^ ((r >> 2) & 3): no bank conflicts on either side.
template <int BM, int BN>
__global__ __launch_bounds__(F32_THREADS, (BM + BN > 192 ? 2 : 3)) void gemm_f32_kernel(int M, int N, int K, const float* __restrict__ A,
    const float* __restrict__ W, const float* __restrict__ bias, int act, float alpha, int out_mode, void* __restrict__ out, int tiles_n,
    int lda, int ldw, KvStore kv)
{
    constexpr int TM = BM / 32, TN = BN / 32;                // 16-row and 16-feature tiles of a wave
    constexpr int RA = BM * 8 / F32_THREADS, RW = BN * 8 / F32_THREADS;      // groups of 4 elements of a thread per operand and step
    constexpr int PA = BM * F32_ROW, PW = BN * F32_ROW;      // bytes of a plane
    extern __shared__ __align__(16) unsigned char lds[];     // A's planes h, m, l, then W's
    int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int wm = wave >> 1, wn = wave & 1;
    // an XCD's workgroups take neighbouring tiles, feature tiles fastest: they share activation rows in its L2
    int total = gridDim.x, pid = blockIdx.x, chunk = total / 8;
    if (pid < chunk * 8) pid = (pid % 8) * chunk + pid / 8;
    int m0 = pid / tiles_n * BM, n0 = pid % tiles_n * BN;

    // rows past the edge repeat the last one; their results are not stored
    const float *src_a[RA], *src_w[RW];
    unsigned dst_a[RA], dst_w[RW];
    auto place = [&](int i) {
        int u = i * F32_THREADS + tid, r = u >> 3, c = u & 7;
        return (unsigned)(r * F32_ROW + (((c >> 1) ^ ((r >> 2) & 3)) << 4) + (c & 1) * 8);
    };
#pragma unroll
    for (int i = 0; i < RA; ++i) {
        int u = i * F32_THREADS + tid, r = m0 + (u >> 3);
        src_a[i] = A + (int64_t)(r < M ? r : M - 1) * lda + (u & 7) * 4;
        dst_a[i] = place(i);
    }
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        int u = i * F32_THREADS + tid, r = n0 + (u >> 3);
        src_w[i] = W + (int64_t)(r < N ? r : N - 1) * ldw + (u & 7) * 4;
        dst_w[i] = 3 * PA + place(i);
    }
    f32x4 va[RA], vw[RW];
    auto fetch = [&](int k) {
#pragma unroll
        for (int i = 0; i < RA; ++i) va[i] = *(const f32x4*)(src_a[i] + k);
#pragma unroll
        for (int i = 0; i < RW; ++i) vw[i] = *(const f32x4*)(src_w[i] + k);
    };
    auto put = [&](f32x4 v, unsigned dst, int plane) {
        uint2 w[3];
        bf16_parts(v * PART_SCALE, w);
#pragma unroll
        for (int p = 0; p < 3; ++p) *(uint2*)(lds + dst + p * plane) = w[p];
    };

    f32x4 acc[TN][TM];
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    int fr = lane & 15, g = lane >> 4;
    const unsigned char* at = lds + fr * F32_ROW + ((g ^ ((fr >> 2) & 3)) << 4);       // rows 16 apart share their swizzle
    const unsigned char *at_a = at + wm * (BM / 2) * F32_ROW, *at_w = at + 3 * PA + wn * (BN / 2) * F32_ROW;

    fetch(0);
    for (int k = 0; k < K; k += F32_BK) {
#pragma unroll
        for (int i = 0; i < RA; ++i) put(va[i], dst_a[i], PA);
#pragma unroll
        for (int i = 0; i < RW; ++i) put(vw[i], dst_w[i], PW);
        __syncthreads();
        if (k + F32_BK < K) fetch(k + F32_BK);
        u32x4 fa[3][TM], fw[2][3];
        auto read_a = [&](int p) {
#pragma unroll
            for (int j = 0; j < TM; ++j) fa[p][j] = *(const u32x4*)(at_a + p * PA + j * 16 * F32_ROW);
        };
        auto read_w = [&](int i, int p) { fw[i & 1][p] = *(const u32x4*)(at_w + p * PW + i * 16 * F32_ROW); };
        // the smallest products first, and their operands
        read_w(0, 2); read_a(0); read_w(0, 0); read_a(2); read_w(0, 1); read_a(1);
#pragma unroll
        for (int i = 0; i < TN; ++i) {
            if (i + 1 < TN) { read_w(i + 1, 2); read_w(i + 1, 0); read_w(i + 1, 1); }
#pragma unroll
            for (int x = 0; x < 6; ++x)
#pragma unroll
                for (int j = 0; j < TM; ++j) acc[i][j] = HalfUnit<bf16_t>::mma(fw[i & 1][PARTS[x][0]], fa[PARTS[x][1]][j], acc[i][j]);
        }
        __syncthreads();
    }

    int row0 = m0 + wm * (BM / 2), col0 = n0 + wn * (BN / 2);
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
        for (int j = 0; j < TM; ++j) {
            // 0 * x is NaN for a sum that is not finite
            f32x4 z = acc[i][j] * 0.f;
            float s = z[0] + z[1] + z[2] + z[3];
            acc[i][j] *= PARTS_UNSCALE;
            if (__builtin_amdgcn_ballot_w64(s != s) == 0) continue;
            int r = row0 + j * 16 + fr, n = col0 + i * 16 + fr;
            const float* pa = A + (int64_t)(r < M ? r : M - 1) * lda + g;
            const float* pw = W + (int64_t)(n < N ? n : N - 1) * ldw + g;
            f32x4 c = {0.f, 0.f, 0.f, 0.f};
            for (int k = 0; k < K; k += 4) c = __builtin_amdgcn_mfma_f32_16x16x4f32(pw[k], pa[k], c, 0, 0, 0);
            acc[i][j] = c;
        }

    unsigned stg = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)lds + wave * 4096;
    if (out_mode == OUT_RESID)
        epilogue_tiles<float, TM, TN, 32, EPI_RESID>(acc, stg, lane, row0, col0, M, N, bias, alpha, (float*)out, nullptr);
    else if (out_mode == OUT_F32)
        epilogue_tiles<float, TM, TN, 32, EPI_F32>(acc, stg, lane, row0, col0, M, N, bias, alpha, (float*)out, nullptr);
    else if (kv.pool)
        epilogue_tiles<float, TM, TN, 32, EPI_T_KV>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (float*)out, kv);
    else if (act == 0)
        epilogue_tiles<float, TM, TN, 32, EPI_T_RELU>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (float*)out);
    else if (act == 1)
        epilogue_tiles<float, TM, TN, 32, EPI_T_GELU>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (float*)out);
    else
        epilogue_tiles<float, TM, TN, 32, EPI_T>(acc, stg, lane, row0, col0, M, N, bias, alpha, nullptr, (float*)out);
}

template <int BM, int BN> static hipError_t launch_f32(const GemmArgs& a, hipStream_t s)
{
    auto kern = gemm_f32_kernel<BM, BN>;
    constexpr int lds = f32_lds(BM, BN);
    static_assert(lds <= 64 * 1024, "no more than a launch takes without asking");
    const int64_t tm = ((int64_t)a.M + BM - 1) / BM, tn = ((int64_t)a.N + BN - 1) / BN, most = MAX_LAUNCH_THREADS / F32_THREADS / tn;
    if (most < 1) return hipErrorInvalidValue;
    const int lda = a.lda ? a.lda : a.K;
    KvStore kv = a.kv ? *a.kv : KvStore{};
    for (int64_t t = 0; t < tm; t += most) {                 // one launch, but for some 10^9 rows
        const int64_t row = t * BM, rows = t + most < tm ? most * BM : a.M - row;
        kern<<<(unsigned)((t + most < tm ? most : tm - t) * tn), F32_THREADS, lds, s>>>((int)rows, a.N, a.K, (const float*)a.A + row * lda, (const float*)a.W,
            (const float*)a.bias, a.act, a.alpha, a.out_mode, (float*)a.out + row * a.N, (int)tn, lda, a.ldw ? a.ldw : a.K, kv);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (kv.pool) {
            kv.row += rows;
            kv.cap += rows;
        }
    }
    return hipSuccess;
}

// The tile, and what a launch takes: n workgroups fall to the busiest CU, `resident` of them at a time (what registers and LDS let in);
// a launch takes `start`, and a step of 32 k takes the resident ones `step` together and each `share` more.  Fitted to 302 shapes on one
// MI355X, 14 weights (256 to 4096 features, K 256 to 4096) x 22 row counts from 32 to 16384: within 1.3, 2.0 and 2.4 % on average (9, 13
// and 12 % at worst), and the tile taken is within 0.2 % of the fastest on average, 8 % at worst.
// us on one MI355X, the float MFMA kernel that this replaces / 128 x 128 / 64 x 128 / 64 x 64, and the 2-norm relative error against
// 64 bits there and here:
//   12288 x  768, K  256  51.2 / 43.2 / 38.0 / 40.3   2.9e-7 2.3e-7     12288 x 1024, K  256  60.9 / 44.5 / 43.5 / 50.7   2.9e-7 2.3e-7
//   12288 x  256, K 1024  57.6 / 61.6 / 57.0 / 50.9   5.7e-7 4.9e-7      8192 x  512, K 2048   163 / 116 / 113 / 124      8.1e-7 7.0e-7
//    3000 x  768, K  256  18.5 / 20.1 / 17.7 / 16.0   2.9e-7 2.3e-7     16384 x 1024, K  256  79.0 / 53.8 / 55.7 / 67.5   2.9e-7 2.3e-7
//    2048 x 1024, K  256  14.5 (streaming kernel) / 19.9 / 14.6 / 12.5     1024 x 4096, K 1024  83.6 (streaming) / 62.8 / 58.1 / 64.8
// The last 128 x 128 step takes 1.1 us per workgroup where its MFMAs alone take 0.7: splitting overlaps with other waves' MFMAs only in
// part.  Two stages in LDS with the splitting between a wave's own MFMAs were slower (8000 x 2048, K 512 103 -> 132).
struct F32Tile { int bm, bn, resident; double start, step, share; };
static const F32Tile F32_TILES[] = {{128, 128, 2, 5.5e-6, 0.90e-6, 0.76e-6}, {64, 128, 4, 3.3e-6, 0.74e-6, 0.48e-6}, {64, 64, 4, 2.7e-6, 0.45e-6, 0.32e-6}};
int gemm_f32_tile(int M, int N, int K, double* seconds)
{
    int best = 0;
    for (int i = 0; i < 3; ++i) {
        const F32Tile& t = F32_TILES[i];
        int64_t tiles = ((int64_t)M + t.bm - 1) / t.bm * (((int64_t)N + t.bn - 1) / t.bn);
        double n = (double)((tiles + 255) / 256), rounds = (double)(((int64_t)n + t.resident - 1) / t.resident);
        double c = t.start + (double)M * N * 4 / 6e12 + (double)(K / F32_BK) * (t.step * rounds + t.share * n);
        if (i == 0 || c < *seconds) {
            *seconds = c;
            best = i;
        }
    }
    return best;
}

double gemm_f32_cost(int M, int N, int K)
{
    double seconds = 0.0;
    gemm_f32_tile(M, N, K, &seconds);
    return seconds;
}

hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s)
{
    double seconds = 0.0;
    switch (gemm_f32_tile(a.M, a.N, a.K, &seconds)) {
        case 0: return launch_f32<128, 128>(a, s);
        case 1: return launch_f32<64, 128>(a, s);
        default: return launch_f32<64, 64>(a, s);
    }
}

}  // namespace exe
