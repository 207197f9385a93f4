// Bandwidth-bound helper kernels: embedding gather, LayerNorm / RMSNorm, K/V append, greedy argmax.
#include "common.h"
#include "kernels.h"

namespace exe {

// V consecutive elements, from storage to float and back
template <typename T, int V> __device__ __forceinline__ void load_f32(const T* p, float (&f)[V])
{
    typedef __attribute__((ext_vector_type(V))) T vec;
    vec v = *(const vec*)p;
#pragma unroll
    for (int i = 0; i < V; ++i) f[i] = to_f32(v[i]);
}
template <typename T, int V> __device__ __forceinline__ void store_f32(T* p, const float (&f)[V])
{
    typedef __attribute__((ext_vector_type(V))) T vec;
    vec v;
#pragma unroll
    for (int i = 0; i < V; ++i) v[i] = from_f32<T>(f[i]);
    *(vec*)p = v;
}
// V of the kernels below: 4 where every row and pointer allows it, else 1
static bool vec4_ok(int dtype, int64_t row, const float* f, const void* a, const void* b = nullptr)
{
    uintptr_t m = dtype == DT_F32 ? 15 : 7;
    return row % 4 == 0 && ((uintptr_t)f & 15) == 0 && ((uintptr_t)a & m) == 0 && ((uintptr_t)b & m) == 0;
}

// ---------------------------------------------------------------- descriptors
// A call's descriptors from pinned host memory to the device.  A kernel in the stream, not a copy command: the copy engine's
// hand-over to the kernels behind it took longer than either.
__global__ void stage_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int n)
{
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
}

hipError_t launch_stage(const void* host, void* dev, size_t bytes, hipStream_t s)
{
    int n = (int)((bytes + 15) / 16);
    if (n <= 0) return hipSuccess;
    stage_kernel<<<(n + 255) / 256, 256, 0, s>>>((const uint4*)host, (uint4*)dev, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------- embedding
// h[t][:] = tok_emb[tokens[t]][:] (+ pos_emb[pos[t]][:]); the residual stream h is float.  One element group per thread: with
// one workgroup per row each of its 20 rounds (d = 5120) waited for memory in turn, 17 us for a single row (now 4).
template <typename T, int V>
__global__ void embed_kernel(const int32_t* __restrict__ tokens, const int32_t* __restrict__ pos, int d,
                             const T* __restrict__ tok_emb, const T* __restrict__ pos_emb, float* __restrict__ h)
{
    int t = blockIdx.x, k = (blockIdx.y * blockDim.x + threadIdx.x) * V;
    if (k >= d) return;
    float v[V], p[V];
    load_f32<T, V>(tok_emb + (int64_t)tokens[t] * d + k, v);
    if (pos_emb) {
        load_f32<T, V>(pos_emb + (int64_t)pos[t] * d + k, p);
#pragma unroll
        for (int i = 0; i < V; ++i) v[i] += p[i];
    }
    store_f32<float, V>(h + (int64_t)t * d + k, v);
}

template <typename T, int V> __global__ void load_hidden_kernel(const T* __restrict__ x, int64_t n, float* __restrict__ h)
{
    int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * V;
    int64_t stride = (int64_t)gridDim.x * blockDim.x * V;
    for (; i < n; i += stride) {
        float v[V];
        load_f32<T, V>(x + i, v);
        store_f32<float, V>(h + i, v);
    }
}

template <typename T, int V> __global__ void store_hidden_kernel(const float* __restrict__ h, int64_t n, T* __restrict__ out)
{
    int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) * V;
    int64_t stride = (int64_t)gridDim.x * blockDim.x * V;
    for (; i < n; i += stride) {
        float v[V];
        load_f32<float, V>(h + i, v);
        store_f32<T, V>(out + i, v);
    }
}

template <typename T, int V>
static hipError_t embed_shape(const int32_t* tokens, const int32_t* pos, int T_, int d, const void* te, const void* pe, float* h, hipStream_t s)
{
    int groups = (d + V - 1) / V, threads = groups >= 256 ? 256 : 64;
    embed_kernel<T, V><<<dim3(T_, (groups + threads - 1) / threads), threads, 0, s>>>(tokens, pos, d, (const T*)te, (const T*)pe, h);
    return hipGetLastError();
}

hipError_t launch_embed(int dtype, const int32_t* tokens, const int32_t* pos, int T, int d, const void* tok_emb,
                        const void* pos_emb, float* h, hipStream_t s)
{
    if (T <= 0) return hipSuccess;
    bool v4 = vec4_ok(dtype, d, h, tok_emb, pos_emb);
    if (dtype == DT_F32) return v4 ? embed_shape<float, 4>(tokens, pos, T, d, tok_emb, pos_emb, h, s) : embed_shape<float, 1>(tokens, pos, T, d, tok_emb, pos_emb, h, s);
    return v4 ? embed_shape<bf16_t, 4>(tokens, pos, T, d, tok_emb, pos_emb, h, s) : embed_shape<bf16_t, 1>(tokens, pos, T, d, tok_emb, pos_emb, h, s);
}

template <typename T, int V> static hipError_t hidden_shape(const void* x, float* h, void* out, int64_t n, hipStream_t s)
{
    int64_t want = (n + 256 * V - 1) / (256 * V);
    int blocks = (int)(want < 8192 ? want : 8192);
    if (x) load_hidden_kernel<T, V><<<blocks, 256, 0, s>>>((const T*)x, n, h);
    else store_hidden_kernel<T, V><<<blocks, 256, 0, s>>>(h, n, (T*)out);
    return hipGetLastError();
}

static hipError_t hidden_any(int dtype, const void* x, float* h, void* out, int64_t n, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    bool v4 = vec4_ok(dtype, n, h, x, out);
    if (dtype == DT_F32) return v4 ? hidden_shape<float, 4>(x, h, out, n, s) : hidden_shape<float, 1>(x, h, out, n, s);
    return v4 ? hidden_shape<bf16_t, 4>(x, h, out, n, s) : hidden_shape<bf16_t, 1>(x, h, out, n, s);
}

hipError_t launch_load_hidden(int dtype, const void* x, int64_t n, float* h, hipStream_t s) { return hidden_any(dtype, x, h, nullptr, n, s); }

hipError_t launch_store_hidden(int dtype, const float* h, int64_t n, void* out, hipStream_t s)
{
    return hidden_any(dtype, nullptr, const_cast<float*>(h), out, n, s);
}

// ---------------------------------------------------------------- norms
// One workgroup per row, the row in registers (Q groups of 4 elements per thread); statistics are exact two-pass in float:
// LayerNorm: mean, then the mean of squared deviations; RMSNorm: mean of squares.
//
// With `partial` the kernel first finishes the product that ends in the residual stream: x += sum of the split-K partials
// (in split order, then the bias), which saves the reduction kernel between a projection and the norm behind it.
//
// What bounds it: few rows are a chain of latencies (loads, two reductions, store), so every load is issued before the
// first reduction; many rows are a stream.  Measured against a kernel that keeps the row in LDS, us per launch:
//   1 x 5120 3.7 -> 3.1, with 4 partials (reduction + norm before) 8.3 -> 4.2; 32 x 5120 with 4 7.4 -> 4.5; 256 x 5120 with 4
//   10.4 -> 5.7; 512 x 5120 with 2 15.3 -> 7.7; 64 x 1024 with 8 5.7 -> 3.0; 16384 x 5120 108 -> 90 (5.6 TB/s);
//   8192 x 1024 16.8 -> 9.8; float 12288 x 256 15.5 -> 6.2
template <int NT> __device__ __forceinline__ float block_sum(float v, float* red)
{
    v = wave_sum(v);
    if (NT == 64) return v;
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < NT / 64; ++i) t += red[i];
    return t;
}

// four consecutive elements (k is a multiple of 4, rows start at multiples of 4 elements) as one access
__device__ __forceinline__ f32x4 load4(const float* p) { return *(const f32x4*)p; }
__device__ __forceinline__ f32x4 load4(const bf16_t* p)
{
    uint2 u = *(const uint2*)p;
    return f32x4{bf16lo(u.x), bf16hi(u.x), bf16lo(u.y), bf16hi(u.y)};
}
__device__ __forceinline__ void store4(float* p, f32x4 v) { *(f32x4*)p = v; }
__device__ __forceinline__ void store4(bf16_t* p, f32x4 v)
{
    bf16x4 w;
#pragma unroll
    for (int j = 0; j < 4; ++j) w[j] = (bf16_t)v[j];
    *(bf16x4*)p = w;
}

template <typename T, bool RMS, int NT, int Q, bool LATE>
__global__ __launch_bounds__(NT) void norm_kernel(float* __restrict__ x, const int32_t* __restrict__ row_index, int d,
                                                  const float* __restrict__ partial, int splits, int64_t slice,
                                                  const T* __restrict__ bias, const T* __restrict__ gain,
                                                  const T* __restrict__ shift, float eps, float out_scale, T* __restrict__ out)
{
    __shared__ float red[2][16];
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    int r = blockIdx.x;
    int64_t src = row_index ? row_index[r] : r;
    float* xr = x + src * d;
    f32x4 v[Q], g[Q], b[Q];
    auto at = [&](int q) { return (q * NT + (int)threadIdx.x) * 4; };
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        int k = at(q);
        v[q] = k < d ? load4(xr + k) : zero;
        g[q] = !LATE && k < d ? load4(gain + k) : zero;
        b[q] = !LATE && !RMS && k < d ? load4(shift + k) : zero;
    }
    if (partial) {
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            int k = at(q);
            if (k >= d) continue;
            const float* p = partial + src * d + k;
            f32x4 sum = load4(p);
            int s = 1;
            for (; s + 3 <= splits; s += 3) {
                f32x4 p0 = load4(p + s * slice), p1 = load4(p + (s + 1) * slice), p2 = load4(p + (s + 2) * slice);
                sum += p0;
                sum += p1;
                sum += p2;
            }
            for (; s < splits; ++s) sum += load4(p + s * slice);
            if (bias) sum += load4(bias + k);
            v[q] += sum;
            store4(xr + k, v[q]);
        }
    }
    float s = 0.f;
#pragma unroll
    for (int q = 0; q < Q; ++q)
        s += RMS ? (v[q].x * v[q].x + v[q].y * v[q].y + v[q].z * v[q].z + v[q].w * v[q].w) : (v[q].x + v[q].y + v[q].z + v[q].w);
    float tot = block_sum<NT>(s, red[0]);
    float mean = 0.f, rstd;
    if (RMS) {
        rstd = 1.f / sqrtf(tot / d + eps);
    } else {
        mean = tot / d;
        float sq = 0.f;
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            float e0 = v[q].x - mean, e1 = v[q].y - mean, e2 = v[q].z - mean, e3 = v[q].w - mean;
            if (at(q) < d) sq += e0 * e0 + e1 * e1 + e2 * e2 + e3 * e3;
        }
        rstd = 1.f / sqrtf(block_sum<NT>(sq, red[1]) / d + eps);
    }
    T* o = out + (int64_t)r * d;
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        int k = at(q);
        if (k >= d) continue;
        f32x4 y, gq = LATE ? load4(gain + k) : g[q], bq = LATE && !RMS ? load4(shift + k) : b[q];
#pragma unroll
        for (int j = 0; j < 4; ++j) y[j] = ((v[q][j] - mean) * rstd * gq[j] + bq[j]) * out_scale;
        store4(o + k, y);
    }
}

template <typename T, bool RMS, int NT, int Q, bool LATE = false> static hipError_t norm_go(const NormArgs& a, hipStream_t s)
{
    norm_kernel<T, RMS, NT, Q, LATE><<<a.rows, NT, 0, s>>>(a.x, a.row_index, a.d, a.partial, a.splits, (int64_t)a.partial_rows * a.d,
                                                     (const T*)a.bias, (const T*)a.gain, (const T*)a.shift, a.eps, a.out_scale,
                                                     (T*)a.out);
    return hipGetLastError();
}

// Launch shape.  Few rows: as many threads as keep a thread at one or two groups, for the latency of the chain.  From 2048
// rows on the chip is full whatever the shape, and small workgroups with more per thread are the faster stream (12288 x 256:
// 64 threads 6.2 us, 256 11.1; 8192 x 1024: 64 threads 9.8 us, 256 13.6; 16384 x 5120: 512 threads 90 us, 1024 123).
// Rows of more than 5120: gain and shift are loaded behind the statistics (LATE).  Held from the start they cost 8 registers per
// group, and with them the waves that hide the stream, or spills from 16384 on.  us per launch, kernel with the row in LDS /
// loaded first / late: LayerNorm bf16 8192 x 12288 129 / 156 / 105, 8192 x 20480 351 / 461 / 181, float 2048 x 16388
// 60 / 125 / 46, 16 x 16388 6.5 / 9.6 / 4.6; float RMSNorm, with one of the four arrays in play, is no faster late.
template <typename T, bool RMS> static hipError_t norm_shape(const NormArgs& a, hipStream_t s)
{
    constexpr bool LATE = !RMS || sizeof(T) == 2;
    int q = a.d / 4;
    bool many = a.rows >= 2048;
    if (q <= 64) return norm_go<T, RMS, 64, 1>(a, s);
    if (q <= 128 && many) return norm_go<T, RMS, 64, 2>(a, s);
    if (q <= 256) return many ? norm_go<T, RMS, 64, 4>(a, s) : norm_go<T, RMS, 256, 1>(a, s);
    if (q <= 512) return norm_go<T, RMS, 256, 2>(a, s);
    if (q <= 1024) return many ? norm_go<T, RMS, 256, 4>(a, s) : norm_go<T, RMS, 512, 2>(a, s);
    if (q <= 1280) return many ? norm_go<T, RMS, 512, 3>(a, s) : norm_go<T, RMS, 640, 2>(a, s);
    if (q <= 2048) return norm_go<T, RMS, 512, 4, LATE>(a, s);
    if (q <= 3072) return norm_go<T, RMS, 768, 4, LATE>(a, s);
    if (q <= 4096) return norm_go<T, RMS, 1024, 4, LATE>(a, s);
    if (q <= 5120) return norm_go<T, RMS, 1024, 5, LATE>(a, s);
    if (q <= 7168) return norm_go<T, RMS, 1024, 7, LATE>(a, s);
    return norm_go<T, RMS, 1024, 9, LATE>(a, s);
}

hipError_t launch_norm(const NormArgs& a, hipStream_t s)
{
    if (a.rows <= 0) return hipSuccess;
    if (a.d % 4 != 0 || a.d > 36864) return hipErrorInvalidValue;
    if (a.dtype == DT_F32) return a.rms ? norm_shape<float, true>(a, s) : norm_shape<float, false>(a, s);
    return a.rms ? norm_shape<bf16_t, true>(a, s) : norm_shape<bf16_t, false>(a, s);
}

// ---------------------------------------------------------------- K/V append
// grid (T, 2): blockIdx.y = 0 keys, 1 values.  Each thread moves 16 bytes.
template <typename T>
__global__ void kv_append_kernel(const T* __restrict__ src, int ld, int k_off, int v_off,
                                 const int32_t* __restrict__ tok_b, const int32_t* __restrict__ tok_pos,
                                 const int64_t* __restrict__ base, const int32_t* __restrict__ cap, int layer, int H,
                                 int dh, T* __restrict__ pool)
{
    constexpr int EPL = 16 / sizeof(T);
    int t = blockIdx.x, kv = blockIdx.y;
    int b = tok_b ? tok_b[t] : t;
    int pos = tok_pos[t];
    int64_t c = cap[b];
    const T* s = src + (int64_t)t * ld + (kv ? v_off : k_off);
    T* dst = pool + base[b] + ((int64_t)(layer * 2 + kv) * H) * c * dh + (int64_t)pos * dh;
    int inner = H * dh;
    for (int e = threadIdx.x * EPL; e < inner; e += blockDim.x * EPL) {
        int head = e / dh, col = e - head * dh;
        *(uint4*)(dst + (int64_t)head * c * dh + col) = *(const uint4*)(s + e);
    }
}

hipError_t launch_kv_append(int dtype, const void* src, int ld, int k_off, int v_off, int T, const int32_t* tok_b,
                            const int32_t* tok_pos, const int64_t* base, const int32_t* cap, int layer, int H, int dh,
                            void* pool, hipStream_t s)
{
    if (T <= 0) return hipSuccess;
    int epl = dtype == DT_F32 ? 4 : 8;
    if (dh % epl || ld % epl || k_off % epl || v_off % epl) return hipErrorInvalidValue;
    dim3 grid(T, 2);
    if (dtype == DT_F32)
        kv_append_kernel<float><<<grid, 256, 0, s>>>((const float*)src, ld, k_off, v_off, tok_b, tok_pos, base, cap,
                                                     layer, H, dh, (float*)pool);
    else
        kv_append_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t*)src, ld, k_off, v_off, tok_b, tok_pos, base,
                                                      cap, layer, H, dh, (bf16_t*)pool);
    return hipGetLastError();
}

__global__ void kv_rows_kernel(const int32_t* __restrict__ tok_b, const int32_t* __restrict__ tok_pos, const int64_t* __restrict__ base,
                               const int32_t* __restrict__ cap, int T, int dh, int64_t* __restrict__ row, int32_t* __restrict__ row_cap)
{
    int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    int b = tok_b[t];
    row[t] = kv_row_of(base[b], tok_pos[t], dh);
    row_cap[t] = cap[b];
}

hipError_t launch_kv_rows(const int32_t* tok_b, const int32_t* tok_pos, const int64_t* base, const int32_t* cap, int T, int dh,
                          int64_t* row, int32_t* row_cap, hipStream_t s)
{
    if (T <= 0) return hipSuccess;
    kv_rows_kernel<<<(T + 255) / 256, 256, 0, s>>>(tok_b, tok_pos, base, cap, T, dh, row, row_cap);
    return hipGetLastError();
}

// Paged pool: the same rows into blocks of 2^shift positions.  `layer_pool` is the layer's slab of blocks, block b at
// b * 2*H*2^shift*dh elements holding [K|V][head][row][dh]; table [sequences][table_w] lists each sequence's blocks.
template <typename T>
__global__ void kv_append_paged_kernel(const T* __restrict__ src, int ld, int k_off, int v_off,
                                       const int32_t* __restrict__ tok_b, const int32_t* __restrict__ tok_pos,
                                       const int32_t* __restrict__ table, int table_w, int shift, int H, int dh,
                                       T* __restrict__ layer_pool)
{
    constexpr int EPL = 16 / sizeof(T);
    int t = blockIdx.x, kv = blockIdx.y;
    int b = tok_b ? tok_b[t] : t;
    int pos = tok_pos[t];
    int64_t rows = (int64_t)1 << shift;
    int blk = table[(int64_t)b * table_w + (pos >> shift)];
    const T* s = src + (int64_t)t * ld + (kv ? v_off : k_off);
    T* dst = layer_pool + ((int64_t)blk * 2 + kv) * H * rows * dh + (int64_t)(pos & (rows - 1)) * dh;
    int inner = H * dh;
    for (int e = threadIdx.x * EPL; e < inner; e += blockDim.x * EPL) {
        int head = e / dh, col = e - head * dh;
        *(uint4*)(dst + (int64_t)head * rows * dh + col) = *(const uint4*)(s + e);
    }
}

hipError_t launch_kv_append_paged(int dtype, const void* src, int ld, int k_off, int v_off, int T, const int32_t* tok_b,
                                  const int32_t* tok_pos, const int32_t* table, int table_w, int shift, int H, int dh,
                                  void* layer_pool, hipStream_t s)
{
    if (T <= 0) return hipSuccess;
    int epl = dtype == DT_F32 ? 4 : 8;
    if (dh % epl || ld % epl || k_off % epl || v_off % epl || !table || table_w < 1) return hipErrorInvalidValue;
    dim3 grid(T, 2);
    if (dtype == DT_F32)
        kv_append_paged_kernel<float><<<grid, 256, 0, s>>>((const float*)src, ld, k_off, v_off, tok_b, tok_pos, table, table_w,
                                                           shift, H, dh, (float*)layer_pool);
    else
        kv_append_paged_kernel<bf16_t><<<grid, 256, 0, s>>>((const bf16_t*)src, ld, k_off, v_off, tok_b, tok_pos, table,
                                                            table_w, shift, H, dh, (bf16_t*)layer_pool);
    return hipGetLastError();
}

// ---------------------------------------------------------------- greedy argmax
// One workgroup per row; ties resolve to the lowest index at every level of the reduction.  D loads in flight per thread: one at
// a time, a row of 50 272 logits took 20 us (with four 7).  `out` may be pinned host memory.
template <int V, unsigned D> __global__ __launch_bounds__(1024) void argmax_kernel(const float* __restrict__ logits, int n, int32_t* __restrict__ out)
{
    __shared__ float bv[16];
    __shared__ int bi[16];
    const float* x = logits + (int64_t)blockIdx.x * n;
    float best = -INFINITY;
    int idx = 0x7fffffff;
    for (unsigned i0 = threadIdx.x * V; i0 < (unsigned)n; i0 += 1024 * V * D) {       // unsigned: i0 runs past n, which may be 2^31 - 1
        float v[D][V];
#pragma unroll
        for (unsigned d = 0; d < D; ++d) {
            unsigned i = i0 + d * 1024 * V;
            load_f32<float, V>(x + (i < (unsigned)n ? i : i0), v[d]);
        }
#pragma unroll
        for (unsigned d = 0; d < D; ++d)
#pragma unroll
            for (int e = 0; e < V; ++e) {
                unsigned i = i0 + d * 1024 * V + e;
                if (i < (unsigned)n && (v[d][e] > best || (v[d][e] == best && (int)i < idx))) { best = v[d][e]; idx = (int)i; }
            }
    }
    if (idx == 0x7fffffff) { best = -INFINITY; }
    argmax_rows(best, idx);
    int w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) { bv[w] = best; bi[w] = idx; }
    __syncthreads();
    if (threadIdx.x < 16) {                      // the 16 waves' candidates, one a lane
        best = bv[threadIdx.x];
        idx = bi[threadIdx.x];
        argmax_row16(best, idx);
    }
    if (threadIdx.x == 0) {
        out[blockIdx.x] = idx == 0x7fffffff ? 0 : idx;
    }
}

hipError_t launch_argmax(const float* logits, int rows, int n, int32_t* out, hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    // rows that one load per thread covers want no more (2000 rows of 100: four loads 12.6 us, one 10.8; of 4096: 16.2 and 13.9)
    if (n % 4 == 0 && ((uintptr_t)logits & 15) == 0) {
        if (n <= 4096) argmax_kernel<4, 1><<<rows, 1024, 0, s>>>(logits, n, out);
        else argmax_kernel<4, 4><<<rows, 1024, 0, s>>>(logits, n, out);
    } else if (n <= 1024) argmax_kernel<1, 1><<<rows, 1024, 0, s>>>(logits, n, out);
    else argmax_kernel<1, 4><<<rows, 1024, 0, s>>>(logits, n, out);
    return hipGetLastError();
}

}  // namespace exe
