// A decode iteration of a small model: attention and feed-forward of a layer as one launch each.
//
// What bounds such an iteration is not its arithmetic or its bytes but the chain of launches, each 3.5 to 5 us of which the
// work is one: waves start, a load or two return from another XCD's writes, a reduction, a store.  Five launches a layer (norm +
// QKV, attention, out-projection, norm + FFN1, FFN2; eight with cross-attention) become two (three), without any waiting between
// workgroups: the work of a launch is cut where one workgroup can carry a piece of it to the end, and what has to be added up
// across workgroups is left as partial sums, which whoever needs the residual stream next adds for itself (as split-K partial
// sums are, see norm_kernel).
//
//   small_attn_kernel   workgroup = (head, row): the row's residual stream and norm, q, k, v of its head, attention over its
//                       cached rows, and the head's share of the out-projection -> partial sums [head][row][d]
//   small_ffn_kernel    workgroup = 32 features of the feed-forward: all rows' residual stream and norm, FFN1 of those features,
//                       activation, their share of FFN2 -> partial sums [slice][row][d]
//
// The residual stream goes back and forth between two buffers: every workgroup of a launch reads the old rows, one of them writes
// the new ones.  Roundings are those of the launches this replaces: norm output, q, k, v, attention output and activations in the
// storage type, everything else float.
//
// Measured on one MI355X, us per decode iteration before -> now (device time by the profiler):
//   float, 2 layers of 256 (4 heads), feed-forward 1024, 4 rows of 8 to 48 cached positions     51 -> 40
//   float, 2 encoder-decoder layers of 256, feed-forward 512, 12 rows, 96 encoder positions      86 -> 64
// and per launch: attention block 8.8 (norm + QKV, attention, out-projection 11.1), cross-attention block 8.4 (14.0), feed-forward
// block 5.8 (8.0).  In the attention block the row with its partial sums arrives after 3 us, the norm takes 0.7, q, k, v and their
// hand-over 1.1, attention and its merge 1.4, the out-projection 0.6, start and end of the launch 2.
#include "attn_row.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace exe {

// what a row of the residual stream is before a block: x (or the embedding) + partial sums in order + their bias
template <typename T> struct SmallRow {
    const float* x;
    const int32_t *tokens, *pos;         // tokens nullable: the row is its embedding, x is not read
    const T *tok_emb, *pos_emb;          // pos_emb nullable
    const float* partial;                // [n_part][rows][d]
    const T* part_bias;                  // nullable
    int n_part;
    float* x_out;                        // where the row goes
    const T *gain, *shift;               // of the block's norm; shift: LayerNorm only
    float eps;
    int rms;
    const uint4* stage_from;             // what the first workgroup of the attention block copies for later launches
    uint4* stage_to;
    int stage_n;
};

constexpr int SA_WAVES = 16, SA_THREADS = SA_WAVES * 64, ATTN_FIRST = 2;     // waves, threads, row blocks in flight per wave
constexpr int SF_WAVES = 8, SF_THREADS = SF_WAVES * 64, SF_F = SMALL_SLICE;

// ---------------------------------------------------------------- attention block
// d * sizeof(T) a multiple of 256, at most 1024 (the weights of three features per lane group stay in registers while the norm is
// computed).  16 lanes share a weight row of q, k, v; the out-projection reads head-wide pieces of W_o's rows as decode attention
// reads keys.
template <typename T, int DH, bool CROSS>
__global__ __launch_bounds__(SA_THREADS) void small_attn_kernel(SmallRow<T> in, int d, int H, const T* __restrict__ w_in, const T* __restrict__ b_in,
                                                                const T* __restrict__ w_out, T* pool, const int64_t* __restrict__ base,
                                                                const int32_t* __restrict__ cap, const int32_t* __restrict__ len,
                                                                const int32_t* __restrict__ qpos, int layer, float scale,
                                                                const float* __restrict__ bias_by_dist, int radius, float* __restrict__ out)
{
    constexpr int EPL = 16 / sizeof(T), CH = 1024 / 256;     // elements of a 16-byte chunk; most chunks of a lane per weight row
    constexpr int NF = CROSS ? DH : 3 * DH, PASSES = NF / 64; // 64 features a pass, 4 per wave
    constexpr int PG = PASSES < 3 ? PASSES : 3;               // passes whose weights are held at once
    constexpr int LPR = DH / EPL, RPW = 64 / LPR;             // lanes per W_o row piece, rows per wave-load
    constexpr int PO = 1024 / sizeof(T) / (SA_WAVES * RPW);   // most wave-loads of W_o
    __shared__ __align__(16) float s_x[512], s_g[512], s_b[512], s_p[SA_THREADS];
    __shared__ __align__(16) T s_qkv[NF], s_ctx[DH];
    int h = blockIdx.x, r = blockIdx.y, rows = gridDim.y, inner = H * DH;
    int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int rg = lane >> 4, cl = lane & 15;
    int chunks = d / (16 * EPL);
    if (h == 0 && r == 0)
        for (int i = tid; i < in.stage_n; i += SA_THREADS) in.stage_to[i] = in.stage_from[i];

    // The partial sums in front go out first, spread over all threads: group tid / d of them takes parts tid / d, + groups, ..
    constexpr int PB = 8;                                     // loads of a thread in flight
    int groups = SA_THREADS / d, grp = tid / d, col = tid - grp * d;
    const float* part = in.partial + (int64_t)r * d + col;
    const int64_t slice = (int64_t)rows * d;
    float pv[PB];
#pragma unroll
    for (int i = 0; i < PB; ++i) {
        int s = grp + i * groups;
        pv[i] = 0.f;
        if (s < in.n_part && grp < groups) pv[i] = part[s * slice];
    }
    float x = 0.f, pb = 0.f, gain = 0.f, shift = 0.f;
    if (tid < d) {
        if (in.tokens) {
            x = to_f32(in.tok_emb[(int64_t)in.tokens[r] * d + tid]);
            if (in.pos_emb) x += to_f32(in.pos_emb[(int64_t)in.pos[r] * d + tid]);
        } else {
            x = in.x[(int64_t)r * d + tid];
        }
        gain = to_f32(in.gain[tid]);
        if (!in.rms) shift = to_f32(in.shift[tid]);
        if (in.part_bias) pb = to_f32(in.part_bias[tid]);
    }
    // then the weights of q, k, v
    uint4 w[PG][CH];
    auto feature = [&](int p) { return p * 64 + wave * 4 + rg; };          // of q, k, v of the head, one behind the other
    auto load_w = [&](int p0) {
#pragma unroll
        for (int p = 0; p < PG; ++p) {
            int f = feature(p0 + p);
            const T* row = w_in + (int64_t)((f / DH) * inner + h * DH + f % DH) * d + cl * EPL;
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (c < chunks) w[p][c] = *(const uint4*)(row + c * 16 * EPL);
        }
    };
    load_w(0);
    float b_own[PASSES];                                      // the biases of the features that this lane stores
#pragma unroll
    for (int p = 0; p < PASSES; ++p) {
        int f = feature(p);
        b_own[p] = b_in ? to_f32(b_in[(f / DH) * inner + h * DH + f % DH]) : 0.f;
    }
    __builtin_amdgcn_sched_barrier(0);
    int64_t kv_at = base[r] + ((int64_t)(layer * 2) * H + h) * cap[r] * DH;
    int64_t kv_size = (int64_t)H * cap[r] * DH;
    int nk = len[r], qp = qpos[r];
    const int table = bias_by_dist ? 2 * radius + 1 : 0;      // the head's bias table, if it fits (see attn_row_body)
    __shared__ float s_bias[ATTN_BIAS_LDS];
    float tb = 0.f;
    if (tid < table && table <= ATTN_BIAS_LDS) tb = bias_by_dist[(int64_t)h * table + tid] * LOG2E;
    if (in.n_part) {                                          // uniform
        float sum = 0.f;
#pragma unroll
        for (int i = 0; i < PB; ++i) sum += pv[i];
        for (int s = grp + PB * groups; s < in.n_part && grp < groups; s += groups) sum += part[s * slice];
        s_p[tid] = sum;
        __syncthreads();
    }
    // the rows of attention's first step arrive during the norm and q, k, v
    EarlyRows<ATTN_FIRST> first;
    {
        constexpr int ROWS = 64 / LPR;
        const int nc = CROSS ? nk : nk - 1, rg_kv = lane / LPR, c_kv = lane % LPR, j0 = wave * ROWS * ATTN_FIRST;
        if (j0 < nc)                                          // uniform in a wave
#pragma unroll
            for (int u = 0; u < ATTN_FIRST; ++u) {
                int row = j0 + u * ROWS + rg_kv;
                const T* kr = pool + kv_at + (int64_t)(row < nc ? row : nc - 1) * DH + c_kv * EPL;
                first.k[u] = load_chunk<true>(kr);
                first.v[u] = load_chunk<true>(kr + kv_size);
            }
    }
    if (tid < d) {
        float sum = pb;
        if (in.n_part)
            for (int i = groups - 1; i >= 0; --i) sum += s_p[i * d + tid];
        x += sum;
        s_x[tid] = x;
        s_g[tid] = gain;
        s_b[tid] = shift;
        if (h == 0) in.x_out[(int64_t)r * d + tid] = x;
    }
    if (tid < table && table <= ATTN_BIAS_LDS) s_bias[tid] = tb;
    __syncthreads();
    // every group of 16 lanes normalises the row for itself: lane cl holds the elements that it multiplies below
    float y[CH][EPL];
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int e = 0; e < EPL; e += 4) {
            f32x4 v = {0.f, 0.f, 0.f, 0.f};
            if (c < chunks) v = *(const f32x4*)&s_x[(c * 16 + cl) * EPL + e];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                y[c][e + i] = v[i];
                sum += in.rms ? v[i] * v[i] : v[i];
            }
        }
    float tot = row_sum<16>(sum), mean = 0.f, var = tot / d;
    if (!in.rms) {
        mean = var;
        float sq = 0.f;
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int e = 0; e < EPL; ++e)
                if (c < chunks) sq += (y[c][e] - mean) * (y[c][e] - mean);
        var = row_sum<16>(sq) / d;
    }
    float rstd = 1.f / sqrtf(var + in.eps);
#pragma unroll
    for (int c = 0; c < CH; ++c)
        if (c < chunks) {
#pragma unroll
            for (int e = 0; e < EPL; e += 4) {
                f32x4 g = *(const f32x4*)&s_g[(c * 16 + cl) * EPL + e], b = *(const f32x4*)&s_b[(c * 16 + cl) * EPL + e];
#pragma unroll
                for (int i = 0; i < 4; ++i) y[c][e + i] = to_f32(from_f32<T>((y[c][e + i] - mean) * rstd * g[i] + b[i]));
            }
        }
#pragma unroll
    for (int p0 = 0; p0 < PASSES; p0 += PG) {
        if (p0 > 0) load_w(p0);
#pragma unroll
        for (int p = 0; p < PG; ++p) {
            float s = 0.f;
#pragma unroll
            for (int c = 0; c < CH; ++c)
                if (c < chunks) {
                    float wf[EPL];
                    Chunk<T, EPL>::unpack(w[p][c], wf);
#pragma unroll
                    for (int e = 0; e < EPL; ++e) s = fmaf(y[c][e], wf[e], s);
                }
            s = row_sum<16>(s);
            if (cl == 0) s_qkv[feature(p0 + p)] = from_f32<T>(s + b_own[p0 + p]);
        }
    }
    // the head's columns of W_o arrive during attention
    uint4 wo[PO];
    int orow = lane / LPR, oc = lane % LPR;
#pragma unroll
    for (int i = 0; i < PO; ++i) {
        int e = (i * SA_WAVES + wave) * RPW + orow;
        if (e < d) wo[i] = *(const uint4*)(w_out + (int64_t)e * inner + h * DH + oc * EPL);
    }
    __syncthreads();
    const T *knew = CROSS ? nullptr : s_qkv + DH, *vnew = CROSS ? nullptr : s_qkv + 2 * DH;
    attn_row_body<T, DH, false, SA_WAVES, ATTN_FIRST, false>(s_qkv, pool + kv_at, pool + kv_at + kv_size, knew, vnew, DH, nk, qp, h, H, scale,
                                                    bias_by_dist, radius, pool, nullptr, 0, s_bias, [&](int c, T o) { s_ctx[c] = o; }, first);
    __syncthreads();
    float cf[EPL];
    Chunk<T, EPL>::unpack(*(const uint4*)&s_ctx[oc * EPL], cf);
#pragma unroll
    for (int i = 0; i < PO; ++i) {
        int e = (i * SA_WAVES + wave) * RPW + orow;
        if ((i * SA_WAVES + wave) * RPW >= d) continue;      // uniform
        float wf[EPL], s = 0.f;
        Chunk<T, EPL>::unpack(wo[i], wf);
#pragma unroll
        for (int k = 0; k < EPL; ++k) s = fmaf(cf[k], wf[k], s);
        s = row_sum<LPR>(s);
        if (oc == 0) out[((int64_t)h * rows + r) * d + e] = s;
    }
}

// ---------------------------------------------------------------- feed-forward block
// Up to MB * 16 rows.  The slice's weights (32 rows of W_1, 32 columns of W_2) go to LDS by direct loads of whole rows while the
// rows are normalised: loaded straight into operand registers, 16 rows a wave-load, they took 3 us of the launch.  Wave
// (tile, quarter) of 2 x 4: 16 of the slice's features, a quarter of K; then every wave a share of FFN2's outputs.
//
// LDS: W_1 and the normed rows, row_bytes and 1024 bytes a row, chunk c (16 bytes) of row r at c ^ (r & 15); W_2 and the
// activations, rows of 32 elements: chunk c of 8 (float) at c ^ ((r >> 1) & 7), of 4 (bf16) at c ^ ((r >> 2) & 3).
constexpr int sf_lds(int MB, int esz) { return 2 * SF_F * 1024 + MB * (16 * 1024 + 3 * 2 * 64 * 16 + 16 * SF_F * esz); }

template <typename T, int MB>
__global__ __launch_bounds__(SF_THREADS) void small_ffn_kernel(SmallRow<T> in, int rows, int d, int f, const T* __restrict__ w_1,
                                                               const T* __restrict__ b_1, int act, const T* __restrict__ w_2,
                                                               float* __restrict__ out)
{
    constexpr int ESZ = sizeof(T);
    constexpr int W2R = SF_F * ESZ, W2C = W2R / 16;          // bytes, chunks of a W_2 row of the slice
    constexpr int U2 = W2R / 64;                             // 64-byte units of it
    constexpr int TO = 1024 / ESZ / 16 / SF_WAVES;           // most 16-feature tiles of a wave in FFN2
    constexpr int QN = 1024 / ESZ / 256;                     // groups of 4 elements per lane and row
    constexpr int RW = MB * 16 / SF_WAVES;                   // rows of a wave
    extern __shared__ __align__(16) unsigned char lds[];
    unsigned char *s_w1 = lds, *s_w2 = s_w1 + SF_F * 1024, *s_a = s_w2 + SF_F * 1024;
    f32x4* s_part = (f32x4*)(s_a + MB * 16 * 1024);          // sums of K's quarters 1 .. 3
    unsigned char* s_u = (unsigned char*)(s_part + 3 * 2 * MB * 64);
    int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int fr = lane & 15, g = lane >> 4, t = wave & 1, kq = wave >> 1;
    int f0 = blockIdx.x * SF_F;
    int row_bytes = d * ESZ;
    auto w2_at = [](int r, int c) { return r * W2R + ((c ^ (W2C == 8 ? (r >> 1) & 7 : (r >> 2) & 3)) << 4); };
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    auto load4 = [](const T* p) {
        typename Vec4<T>::type x = *(const typename Vec4<T>::type*)p;
        return f32x4{to_f32((T)x[0]), to_f32((T)x[1]), to_f32((T)x[2]), to_f32((T)x[3])};
    };

    // rows wave, wave + 8, ..: their residual stream and the first parts to add to it, ahead of the weights
    constexpr int PB = 4;
    const int64_t slice = (int64_t)rows * d;
    f32x4 v[RW][QN], pv[PB][RW][QN], gn[QN], sh[QN], pb[QN];
#pragma unroll
    for (int q = 0; q < QN; ++q) {
        int k = (q * 64 + lane) * 4;
        gn[q] = sh[q] = pb[q] = zero;
#pragma unroll
        for (int i = 0; i < RW; ++i) {
            int r = i * SF_WAVES + wave;
            v[i][q] = zero;
            if (r < rows && k < d) v[i][q] = *(const f32x4*)(in.x + (int64_t)r * d + k);
#pragma unroll
            for (int s = 0; s < PB; ++s) {
                pv[s][i][q] = zero;
                if (s < in.n_part && r < rows && k < d) pv[s][i][q] = *(const f32x4*)(in.partial + s * slice + (int64_t)r * d + k);
            }
        }
        if (k < d) {
            gn[q] = load4(in.gain + k);
            if (!in.rms) sh[q] = load4(in.shift + k);
            if (in.part_bias) pb[q] = load4(in.part_bias + k);
        }
    }
    // 1 KB wave-loads; lane l fills the 16 bytes at l of them with the chunk that belongs there
    typedef __attribute__((address_space(1))) const void* gptr;
    typedef __attribute__((address_space(3))) void* lptr;
    for (int i = wave; i < SF_F * row_bytes / 1024; i += SF_WAVES) {
        int o = i * 1024 + lane * 16, r = o / row_bytes, slot = (o - r * row_bytes) >> 4, c = slot ^ (r & 15);
        __builtin_amdgcn_global_load_lds((gptr)((const unsigned char*)(w_1 + (int64_t)(f0 + r) * d) + c * 16), (lptr)(s_w1 + i * 1024), 16, 0, 0);
    }
    for (int i = wave; i < d * W2R / 1024; i += SF_WAVES) {
        int o = i * 1024 + lane * 16, r = o / W2R, slot = (o % W2R) >> 4, c = slot ^ (W2C == 8 ? (r >> 1) & 7 : (r >> 2) & 3);
        __builtin_amdgcn_global_load_lds((gptr)((const unsigned char*)(w_2 + (int64_t)r * f + f0) + c * 16), (lptr)(s_w2 + i * 1024), 16, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RW; ++i) {
        int r = i * SF_WAVES + wave;
        float s = 0.f;
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            int k = (q * 64 + lane) * 4;
            f32x4 add = pv[0][i][q];
#pragma unroll
            for (int p = 1; p < PB; ++p) add += pv[p][i][q];
            if (r < rows && k < d) {
                const float* p = in.partial + (int64_t)r * d + k;
                for (int j = PB; j < in.n_part; ++j) add += *(const f32x4*)(p + j * slice);
                v[i][q] += add + pb[q];
                if (blockIdx.x == 0) *(f32x4*)(in.x_out + (int64_t)r * d + k) = v[i][q];
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) s += in.rms ? v[i][q][j] * v[i][q][j] : v[i][q][j];
        }
        float tot = wave_sum(s), mean = 0.f, var = tot / d;
        if (!in.rms) {
            mean = var;
            float sq = 0.f;
#pragma unroll
            for (int q = 0; q < QN; ++q)
                if ((q * 64 + lane) * 4 < d)
#pragma unroll
                    for (int j = 0; j < 4; ++j) sq += (v[i][q][j] - mean) * (v[i][q][j] - mean);
            var = wave_sum(sq) / d;
        }
        float rstd = 1.f / sqrtf(var + in.eps);
#pragma unroll
        for (int q = 0; q < QN; ++q) {
            int k = (q * 64 + lane) * 4, byte = k * ESZ;
            if (k >= d) continue;
            typename Vec4<T>::type y;
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = from_f32<T>((v[i][q][j] - mean) * rstd * gn[q][j] + sh[q][j]);
            *(typename Vec4<T>::type*)(s_a + r * 1024 + (((byte >> 4) ^ (r & 15)) << 4) + (byte & 15)) = y;
        }
    }
    __builtin_amdgcn_s_waitcnt(0x0070 | (15 << 8));          // vmcnt(0): this wave's share of the weights has landed
    __syncthreads();

    f32x4 acc[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) acc[m] = zero;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        if (u >= row_bytes / 256) continue;
        int c = (kq * (row_bytes / 256) + u) * 4 + g;
        u32x4 w = *(const u32x4*)(s_w1 + (t * 16 + fr) * row_bytes + ((c ^ fr) << 4));
#pragma unroll
        for (int m = 0; m < MB; ++m) acc[m] = HalfUnit<T>::mma(w, *(const u32x4*)(s_a + (m * 16 + fr) * 1024 + ((c ^ fr) << 4)), acc[m]);
    }
    if (kq) {
#pragma unroll
        for (int m = 0; m < MB; ++m) s_part[(((kq - 1) * 2 + t) * MB + m) * 64 + lane] = acc[m];
    }
    __syncthreads();
    if (!kq) {
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            f32x4 s = acc[m];
#pragma unroll
            for (int q = 0; q < 3; ++q) s += s_part[((q * 2 + t) * MB + m) * 64 + lane];
            if (b_1) s += load4(b_1 + f0 + t * 16 + 4 * g);
            typename Vec4<T>::type y;
#pragma unroll
            for (int j = 0; j < 4; ++j) y[j] = from_f32<T>(act_apply(s[j], act));
            int byte = (t * 16 + 4 * g) * ESZ;
            *(typename Vec4<T>::type*)(s_u + w2_at(m * 16 + fr, byte >> 4) + (byte & 15)) = y;
        }
    }
    __syncthreads();
    u32x4 a[MB][U2];
#pragma unroll
    for (int m = 0; m < MB; ++m)
#pragma unroll
        for (int u = 0; u < U2; ++u) a[m][u] = *(const u32x4*)(s_u + w2_at(m * 16 + fr, u * 4 + g));
#pragma unroll
    for (int i = 0; i < TO; ++i) {
        int e = (i * SF_WAVES + wave) * 16;
        if (e >= d) continue;
#pragma unroll
        for (int m = 0; m < MB; ++m) {
            f32x4 s = zero;
#pragma unroll
            for (int u = 0; u < U2; ++u) s = HalfUnit<T>::mma(*(const u32x4*)(s_w2 + w2_at(e + fr, u * 4 + g)), a[m][u], s);
            int r = m * 16 + fr;
            if (r < rows) *(f32x4*)(out + ((int64_t)blockIdx.x * rows + r) * d + e + 4 * g) = s;
        }
    }
}

// ---------------------------------------------------------------- host side
// Rows of up to 1 KB of weights: what the attention block holds in registers.  Its workgroups each read their head's weights, so
// many rows of many heads cost more than the launches they save: decode iterations of two layers before -> now, us, at rows x heads
// x head size x width of 2M 85 -> 68 and 92 -> 87 (16 rows, float 256 wide; 8, bf16 512 wide, 8 heads), 3.1M 86 -> 86 (12, bf16 512 wide),
// 4.2M 86 -> 89 (16 of those), 93 -> 80 (16, float 256 wide, 16 heads), 6.3M 107 -> 114 (24 of those), 8.4M 101 -> 111.
constexpr int64_t SMALL_MAX_WORK = 3 << 20;
bool small_decode_fits(int dtype, int rows, int d, int H, int dh, int f)
{
    int row_bytes = d * (dtype == DT_F32 ? 4 : 2);
    return rows >= 1 && rows <= SMALL_MAX_ROWS && row_bytes % 256 == 0 && row_bytes <= 1024 && (dh == 64 || dh == 128) &&
           (int64_t)rows * H * dh * d <= SMALL_MAX_WORK && H <= SMALL_MAX_PARTS && f % SF_F == 0 && f / SF_F <= SMALL_MAX_PARTS;
}

template <typename T> static SmallRow<T> small_row(const SmallArgs& a)
{
    return SmallRow<T>{a.x, a.tokens, a.pos, (const T*)a.tok_emb, (const T*)a.pos_emb, a.partial, (const T*)a.part_bias, a.n_part, a.x_out,
                       (const T*)a.gain, (const T*)a.shift, a.eps, a.rms, (const uint4*)a.stage_from, (uint4*)a.stage_to,
                       (int)((a.stage_bytes + 15) / 16)};
}

template <typename T, int DH> static hipError_t small_attn(const SmallArgs& a, const SmallAttn& k, hipStream_t s)
{
    dim3 grid(k.H, a.rows);
#define EXE_SMALL_ATTN(CROSS)                                                                                                            \
    small_attn_kernel<T, DH, CROSS><<<grid, SA_THREADS, 0, s>>>(small_row<T>(a), a.d, k.H, (const T*)k.w_in, (const T*)k.b_in,           \
                                                                (const T*)k.w_out, (T*)k.pool, k.base, k.cap, k.len, k.qpos, k.layer,    \
                                                                k.scale, k.bias_by_dist, k.bias_radius, a.out)
    if (k.cross) EXE_SMALL_ATTN(true);
    else EXE_SMALL_ATTN(false);
#undef EXE_SMALL_ATTN
    return hipGetLastError();
}

hipError_t launch_small_attn(const SmallArgs& a, const SmallAttn& k, hipStream_t s)
{
    if (!small_decode_fits(a.dtype, a.rows, a.d, k.H, k.dh, SF_F)) return hipErrorInvalidValue;
    if (a.dtype == DT_F32) return k.dh == 64 ? small_attn<float, 64>(a, k, s) : small_attn<float, 128>(a, k, s);
    return k.dh == 64 ? small_attn<bf16_t, 64>(a, k, s) : small_attn<bf16_t, 128>(a, k, s);
}

template <typename T> static hipError_t small_ffn(const SmallArgs& a, const SmallFfn& k, hipStream_t s)
{
    static_assert(sf_lds(2, sizeof(T)) <= 160 * 1024, "LDS budget");
    static LdsLimit limit[2][MAX_DEVICES];
    const int mb = a.rows <= 16 ? 1 : 2;
    auto kern = mb == 1 ? small_ffn_kernel<T, 1> : small_ffn_kernel<T, 2>;
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
    hipError_t e = limit[mb - 1][dev].raise((const void*)kern, sf_lds(mb, sizeof(T)));
    if (e != hipSuccess) return e;
    kern<<<k.f / SF_F, SF_THREADS, sf_lds(mb, sizeof(T)), s>>>(small_row<T>(a), a.rows, a.d, k.f, (const T*)k.w_1, (const T*)k.b_1, k.act, (const T*)k.w_2, a.out);
    return hipGetLastError();
}

hipError_t launch_small_ffn(const SmallArgs& a, const SmallFfn& k, hipStream_t s)
{
    if (!small_decode_fits(a.dtype, a.rows, a.d, 1, 64, k.f) || !a.x || a.tokens || !a.partial) return hipErrorInvalidValue;
    return a.dtype == DT_F32 ? small_ffn<float>(a, k, s) : small_ffn<bf16_t>(a, k, s);
}

}  // namespace exe
