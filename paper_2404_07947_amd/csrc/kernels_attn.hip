// Attention kernels.
//
//  * attn_row_kernel<T, DH, PACKED>: one workgroup per (query row, head) streams that row's keys and values
//    with 16-byte loads, float dot products reduced over the lanes that share a key row, and an online
//    softmax whose partial results are merged across the workgroup at the end.
//      PACKED = false: decode / cross attention -- keys and values come from a sequence's cache extent
//                      ([head][capacity][dh] per layer, keys then values).  HBM-bandwidth bound.
//      PACKED = true : ragged prefill, queries from the packed qkv activations, keys and values from there or (base given)
//                      from the cache, for batches of little work (float, and
//                      bf16 with head size 64) and for what the MFMA kernel below does not take (bias tables beyond its
//                      LDS copy, sequences beyond 32-bit offsets).
//  * prefill_mfma_kernel<T, DH, CAUSAL, BIAS>: flash-style ragged prefill.  A workgroup
//    owns 128 query rows of one (sequence, head); keys/values go through LDS in tiles of 64.
//    S^T = K.Q^T and O^T = V^T.P^T are both computed with MFMA 16x16 tiles so that softmax statistics of a
//    query live in the lanes of one accumulator column and P feeds the second MFMA straight from the first
//    one's accumulators.
#include <stdio.h>

#include <algorithm>
#include <mutex>
#include <type_traits>
#include <vector>

#include "attn_row.h"
#include "gemm_epilogue.h"
#include "kernels.h"

namespace exe {

constexpr int ATTN_U = 2;                 // decode attention: row blocks in flight per wave
constexpr int ATTN_LONG_BYTES = 256 << 10;
constexpr int ATTN_LONG_LDS = 88 << 10;   // dynamic LDS that leaves room for one workgroup on a CU

// PAGED (with PACKED = false): the cache of a sequence is a list of blocks of 2^block_shift positions instead of
// one extent.  Block b of the pool holds [K|V][head][position in block][DH]; block_table[r * max_blocks + i] is the
// block with positions i * 2^block_shift .. of sequence r.  The rows of one load of a wave (RPW <= 8 consecutive
// rows starting at a multiple of RPW) never straddle a block (block_shift >= 3).  The RPW * U rows of a whole step
// do not either when RPW * U <= 8: then one table look-up per wave and step suffices; otherwise (bf16, head size
// 64: 16 rows per step) every load of the step has a look-up of its own.
template <typename T, int DH, bool PACKED, int NWV = 4, int U = 4, bool PAGED = false>
__global__ __launch_bounds__(NWV * 64) void attn_row_kernel(
    const T* __restrict__ q, int q_stride, const T* kvbuf, const int64_t* __restrict__ base,
    const int32_t* __restrict__ cap, const int32_t* __restrict__ len, const int32_t* __restrict__ qpos_arr,
    const int32_t* __restrict__ tok_b, const int32_t* __restrict__ cu, int layer, int H, int causal, float scale,
    const float* __restrict__ bias_by_dist, int radius, T* __restrict__ out, int new_k_off, int new_v_off,
    const int32_t* __restrict__ block_table = nullptr, int max_blocks = 0, int block_shift = 0)
{
    static_assert(!(PAGED && PACKED), "paged mode is a cache mode");
    int h = blockIdx.x, r = blockIdx.y;
    int inner = H * DH;

    const T *kp, *vp, *qp;
    int64_t row_stride;
    int nk, qpos;
    if (PACKED) {
        int sb = tok_b[r];
        int t0 = cu[sb];
        qpos = qpos_arr[r];
        nk = causal ? qpos + 1 : cu[sb + 1] - t0;
        row_stride = 3 * (int64_t)inner;
        qp = q + (int64_t)r * row_stride + h * DH;
        if (base) {                          // from the cache, else from the packed activations
            row_stride = DH;
            kp = kvbuf + base[sb] + ((int64_t)(layer * 2) * H + h) * cap[sb] * DH;
            vp = kp + (int64_t)H * cap[sb] * DH;
        } else {
            kp = q + (int64_t)t0 * row_stride + inner + h * DH;
            vp = kp + inner;
        }
    } else if (PAGED) {
        nk = len[r];
        qpos = qpos_arr[r];
        row_stride = DH;
        kp = vp = kvbuf;                    // set per block below
        qp = q + (int64_t)r * q_stride + h * DH;
    } else {
        int64_t c = cap[r];
        nk = len[r];
        qpos = qpos_arr[r];
        row_stride = DH;
        kp = kvbuf + base[r] + ((int64_t)(layer * 2) * H + h) * c * DH;
        vp = kp + (int64_t)H * c * DH;
        qp = q + (int64_t)r * q_stride + h * DH;
    }
    const T *knew = !PACKED && new_k_off ? qp + new_k_off : nullptr, *vnew = !PACKED && new_k_off ? qp + new_v_off : nullptr;
    __shared__ float s_bias[ATTN_BIAS_LDS];
    attn_row_body<T, DH, PACKED, NWV, U, PAGED>(qp, kp, vp, knew, vnew, row_stride, nk, qpos, h, H, scale, bias_by_dist, radius, kvbuf,
                                                PAGED ? block_table + (int64_t)r * max_blocks : nullptr, block_shift, s_bias,
                                                [&](int c, T o) { out[(int64_t)r * inner + h * DH + c] = o; });
}

// Launch shape of a decode attention launch, 2 row blocks in flight per wave (measured best of a sweep over {1,2,3,4,8}), from the
// mean and the largest number of cached rows per sequence (0 = unknown) and the number of workgroups, one per (sequence, head).
//  * 16 waves, fewer where the rows would leave some without a step: 8 up to 16 steps, 4 up to 4, or to 8 where the launch has
//    more workgroups than two per CU and their number hides latencies (256 x 40 heads of 40 rows x 128: 4 waves 42, 8 49, 16 70 us;
//    of 100 rows: 89, 86, 102; 17 heads of 300 x 64: 13.0, 11.6, 11.6).  Just above 512 workgroups of equal rows, a second round of
//    two per CU is nearly empty and small workgroups spread better: 13 x 40 of 256 rows 16.5, 17.1, 17.2 us.
//  * Long streams of different lengths run one workgroup per CU (dynamic LDS that nothing uses keeps a second one out): with two,
//    twice as many streams are open in memory.  Lengths with a standard deviation of a quarter: 1.03 to 1.1x from 256 KB of keys
//    and values on; equal lengths: 0.9x at 256 KB, where two workgroups side by side end together, 0.96 to 1.0x at 512 KB (but 1.04 to
//    1.07x with 4000 workgroups and more), 1.03x from 1 MB on.
struct AttnShape { int waves; bool one_per_cu; };
template <typename T, int DH> static AttnShape attn_shape(int mean_len, int max_len, int64_t wgs)
{
    constexpr int step = 64 / (DH / (16 / (int)sizeof(T))) * ATTN_U;         // rows that a wave takes at a time
    if (mean_len <= 0) return {16, false};
    bool equal = max_len > 0 && (int64_t)max_len * 8 <= (int64_t)mean_len * 9;
    if (mean_len <= (wgs > 512 ? 8 : 4) * step) return {4, false};
    if (mean_len <= 16 * step) return {8, false};
    if (equal && wgs > 512 && wgs <= 640 && mean_len <= 80 * step) return {4, false};
    int64_t bytes = (int64_t)mean_len * 2 * DH * (int)sizeof(T);
    return {16, bytes >= (!equal ? ATTN_LONG_BYTES : wgs >= 2048 ? 2 * ATTN_LONG_BYTES : 4 * ATTN_LONG_BYTES)};
}

template <typename T, int DH, bool PAGED, typename... Args>
static hipError_t launch_attn_row(int mean_len, int max_len, dim3 grid, hipStream_t s, Args... args)
{
    auto k16 = attn_row_kernel<T, DH, false, 16, ATTN_U, PAGED>;
    AttnShape shape = attn_shape<T, DH>(mean_len, max_len, (int64_t)grid.x * grid.y);
    switch (shape.waves) {
        case 4: attn_row_kernel<T, DH, false, 4, ATTN_U, PAGED><<<grid, 256, 0, s>>>(args...); break;
        case 8: attn_row_kernel<T, DH, false, 8, ATTN_U, PAGED><<<grid, 512, 0, s>>>(args...); break;
        default: {
            static LdsLimit limit[MAX_DEVICES];
            int dev = 0;
            if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
            hipError_t e = limit[dev].raise((const void*)k16, ATTN_LONG_LDS);
            if (e != hipSuccess) return e;
            k16<<<grid, 1024, shape.one_per_cu ? ATTN_LONG_LDS : 0, s>>>(args...);
        }
    }
    return hipGetLastError();
}

template <typename T, int DH> static hipError_t launch_attn_cache_t(const AttnCacheArgs& a, hipStream_t s)
{
    const int32_t* none = nullptr;
    return launch_attn_row<T, DH, false>(a.mean_len, a.max_len, dim3(a.H, a.B), s, (const T*)a.q, a.q_stride, (const T*)a.pool, a.base, a.cap, a.len,
                                         a.qpos, none, none, a.layer, a.H, 0, a.scale, a.bias_by_dist, a.bias_radius, (T*)a.out,
                                         a.new_k_off, a.new_v_off, none, 0, 0);
}

hipError_t launch_attn_cache(const AttnCacheArgs& a, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    if (a.dtype == DT_F32 && a.dh == 64) return launch_attn_cache_t<float, 64>(a, s);
    if (a.dtype == DT_F32 && a.dh == 128) return launch_attn_cache_t<float, 128>(a, s);
    if (a.dtype == DT_BF16 && a.dh == 64) return launch_attn_cache_t<bf16_t, 64>(a, s);
    if (a.dtype == DT_BF16 && a.dh == 128) return launch_attn_cache_t<bf16_t, 128>(a, s);
    return hipErrorInvalidValue;
}

// Host-side replay of the paged kernel's row indexing for one sequence of `len` cached rows (the rows a launch with
// these parameters reads, through the same index functions): every row read must be a cached row, lie inside the
// block its look-up names, and every cached row must be read exactly once by an unclamped lane.  Returns 0, or the
// number of violations.
int paged_index_check(int dtype, int dh, int block_shift, int nwv, int len)
{
    int epl = dtype == DT_F32 ? 4 : 8, lpr = dh / epl, rpw = 64 / lpr;
    constexpr int U = ATTN_U;
    int nl = rpw * U > 8 ? U : 1, block_rows = 1 << block_shift, bad = 0;
    if (len < 1 || rpw > 8) return -1;
    int n_blocks = (len + block_rows - 1) >> block_shift;
    std::vector<int> seen(len, 0);
    for (int wave = 0; wave < nwv; ++wave)
        for (int j0 = wave * rpw * U; j0 < len; j0 += nwv * rpw * U)
            for (int u = 0; u < U; ++u) {
                int x = nl == 1 ? 0 : u;
                int lrow = paged_lookup_row(j0, x, rpw, len);
                int entry = lrow >> block_shift, first = lrow & ~(block_rows - 1);
                if (entry < 0 || entry >= n_blocks) ++bad;
                for (int rg = 0; rg < rpw; ++rg) {
                    int row = paged_lane_row(j0, u, rg, rpw, len), in_block = row - first;
                    if (row < 0 || row >= len || in_block < 0 || in_block >= block_rows) ++bad;
                    if (j0 + u * rpw + rg < len) seen[row] += 1;
                }
            }
    for (int r = 0; r < len; ++r)
        if (seen[r] != 1) ++bad;
    return bad;
}

template <typename T, int DH> static hipError_t launch_attn_paged_t(const AttnPagedArgs& a, hipStream_t s)
{
    const int32_t* none = nullptr;
    const int64_t* none64 = nullptr;
    return launch_attn_row<T, DH, true>(a.mean_len, a.max_len, dim3(a.H, a.B), s, (const T*)a.q, a.q_stride, (const T*)a.pool, none64, none, a.len,
                                        a.qpos, none, none, 0, a.H, 0, a.scale, a.bias_by_dist, a.bias_radius, (T*)a.out,
                                        a.new_k_off, a.new_v_off, a.block_table, a.max_blocks, a.block_shift);
}

hipError_t launch_attn_paged(const AttnPagedArgs& a, hipStream_t s)
{
    if (a.B <= 0) return hipSuccess;
    if (a.block_shift < 3 || a.block_shift > 12 || a.max_blocks < 1) return hipErrorInvalidValue;
    if (a.dtype == DT_F32 && a.dh == 64) return launch_attn_paged_t<float, 64>(a, s);
    if (a.dtype == DT_F32 && a.dh == 128) return launch_attn_paged_t<float, 128>(a, s);
    if (a.dtype == DT_BF16 && a.dh == 64) return launch_attn_paged_t<bf16_t, 64>(a, s);
    if (a.dtype == DT_BF16 && a.dh == 128) return launch_attn_paged_t<bf16_t, 128>(a, s);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------- MFMA prefill (described for bf16, head size 128)
// A workgroup of 4 waves owns PREFILL_TILE_Q = 128 query rows of one (sequence, head), 32 per wave as two 16-row
// blocks (QB = 1: 64 rows, one block per wave); three workgroups fit a CU (48 KB of LDS each and the bias table, at most 168
// registers).  Keys and values pass through LDS in tiles of 64 rows (two key tiles, double buffered, and one value tile, or V2:
// two), both by direct global->LDS loads in the same row-major swizzled layout.  Per tile a wave computes
//   S^T[key][query] = K . Q^T      (MFMA 16x16x32: A = key rows from LDS, B = the wave's query fragments)
//   O^T[d][query]  += V^T . P^T    (A = values through the transposing LDS read, B = P straight from the
//                                   accumulators of S^T)
// so a query's softmax statistics live in the four lanes that share its column, and the probabilities never leave
// registers.  Two barriers per tile (the value tile is loaded behind the scores; V2: one).  The workgroups of a CU drift
// apart, so one wave's softmax (vector ALU) overlaps another's MFMAs on the same SIMD.
constexpr int PF_BIAS = 1024, PF_BIAS_PAD = 96;                  // entries of a head's bias table in LDS, and of its continuation on either side
constexpr int pf_bias_entries(int radius) { return 2 * (radius + PF_BIAS_PAD) + 1; }
constexpr int PF_NW = 4, PF_KT = PREFILL_TILE_K, PF_THREADS = PF_NW * 64, PF_QT = PF_NW * 32;
static_assert(PF_QT == PREFILL_TILE_Q, "the tile list is built for PREFILL_TILE_Q query rows per workgroup");
constexpr int pf_tile_bytes(int row_bytes) { return PF_KT * row_bytes; }
template <typename T, int DH, bool V2> constexpr int pf_lds()     // two key tiles, then the value tile(s)
{
    return (V2 ? 4 : 3) * pf_tile_bytes(DH * (int)sizeof(T));
}
// float x 64: three bf16 parts per key, value, query and probability, the parts of one key and one value tile in LDS
template <typename T, int DH> constexpr bool pf_parted() { return sizeof(T) == 4 && DH == 64; }
// workgroups per CU that the registers must leave room for (LDS does)
template <typename T, int DH, bool V2> constexpr int pf_per_cu()
{
    if (sizeof(T) == 4) return DH == 128 ? 1 : 3;
    return DH == 64 ? 5 : V2 ? 2 : 3;
}

// A key or value tile [64 rows] in LDS, row-major in 16-byte chunks.  Rows of 256 bytes and more keep chunk c of row r at
// slot c ^ (r & 15), rows of 128 bytes at slot c ^ ((r >> 1) & 7): the fragment reads below touch every bank group
// equally.  Rows 16 apart share their swizzle.
template <int RB> __device__ __forceinline__ int pf_swz(int row) { return RB >= 256 ? row & 15 : (row >> 1) & 7; }

typedef __attribute__((ext_vector_type(4))) short pf_v4s;
// Transposing LDS read (ds_read_b64_tr_b16).  Within each block of 16 lanes, lane L points at 4 consecutive 16-bit
// elements M[L][0..3]; lane i receives M[4*j + i/4][i%4], j = 0..3.  With lane L = 4*j + q pointing at columns
// d0 + 4*q .. +3 of row j, lane i ends up with column d0 + i of rows 0..3: four values along the row index for one
// column, which is how an MFMA operand wants a row-major tile whose rows are the contraction index.
__device__ __forceinline__ uint2 pf_read_tr(const unsigned char* p)
{
    pf_v4s r = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) pf_v4s*)p);
    return __builtin_bit_cast(uint2, r);
}

// One query row q by one wave, keys 0 .. nk - 1 in order, 64 at a time: a lane takes a key for the scores, and features lane,
// lane + 64 of the result.  ld: elements between rows of keys and values; sc: the scale for exp2.
template <typename T, int DH, bool BIAS>
__device__ __forceinline__ void prefill_row(const T* q, const T* keys, const T* values, int64_t ld, int qr, int nk, float sc,
                                            const float* sbias, int radius, int lane, T* out)
{
    float m = -INFINITY, l = 0.f, acc[DH / 64] = {};
    for (int j0 = 0; j0 < nk; j0 += 64) {
        int j = j0 + lane, cnt = nk - j0 < 64 ? nk - j0 : 64;
        const T* k = keys + (j < nk ? j : nk - 1) * ld;
        float s = 0.f;
#pragma unroll 4
        for (int e = 0; e < DH; ++e) s = fmaf(to_f32(q[e]), to_f32(k[e]), s);
        s *= sc;
        if (BIAS) {
            int rel = j - qr;
            s += sbias[(rel < -radius ? -radius : (rel > radius ? radius : rel)) + radius];
        }
        if (j >= nk) s = -INFINITY;
        float mx = wave_max(fmaxf(m, s)), mref = mx == -INFINITY ? 0.f : mx;
        float alpha = fast_exp2(m - mref), p = fast_exp2(s - mref);
        l = l * alpha + wave_sum(p);
#pragma unroll
        for (int f = 0; f < DH / 64; ++f) acc[f] *= alpha;
        for (int t = 0; t < cnt; ++t) {
            float pt = __shfl(p, t, WAVE);
            const T* v = values + (j0 + t) * ld + lane;
#pragma unroll
            for (int f = 0; f < DH / 64; ++f) acc[f] = fmaf(pt, to_f32(v[f * 64]), acc[f]);
        }
        m = mx;
    }
#pragma unroll
    for (int f = 0; f < DH / 64; ++f) out[lane + f * 64] = from_f32<T>(acc[f] / l);
}

// Head size 64: half the bytes per tile, so the value tiles are double buffered too.  Its probabilities enter the second
// product as the sum of three bf16 values, their first, second and third 8 bits, so no bit of the float is lost (from 2^-110 on; below,
// bf16 holds fewer of them): the row kernel, which served this head size before, multiplies floats too.  The two further sets of
// MFMAs hide behind the exponentials for the most part (one set more and a rounded rest, 2^-17 relative: 40 us where three
// take 43).
//
// Float x 64: bf16 MFMAs too, six for the products that count of three bf16 parts per float (see kernels_gemm_f32.hip), in 3/8
// of the time that eight float MFMAs take.  Keys and values are parted by all threads on their way through registers into
// LDS, one tile of either; the next tile's loads are in flight meanwhile.  A score, and a tile's share of an output, is the sum
// of three numbers: the first parts' products of 32 features (keys) twice, and all the others'.  Error against 64 bits, 2-norm
// relative, float MFMAs / row kernel / now: 200 rows 1.22e-7 / 1.09e-7 / 1.05e-7, 1000 1.38e-7 / 1.31e-7 / 1.20e-7, inputs three times
// as large 3.95e-7 / 3.98e-7 / 3.71e-7, 4096 rows 1.62e-7 / 1.71e-7 / 1.45e-7; in one chain of additions 1.71e-7 at 1000.  Parts are of
// the values times PART_SCALE (see bf16_parts), so that small ones keep all of their bits, probabilities too.  What the parts or the
// sums cannot hold (infinities, NaN, values of 2^104, scores and sums of 2^80 and more) makes NaN, and such rows are computed again.
//
// Float x 128: the same tiles and softmax with 16x16x4 MFMAs, four per 16-byte fragment; the second product takes one key per lane
// group and MFMA, so P again goes from accumulator to operand without moving, and V is read 4 bytes per lane.  A score is the
// pairwise sum of sums of 8 features, an output of sums over 16 keys: with one chain of additions for either, the kernel erred
// 2.3 to 3.3 times as much against 64 bits as the row kernel, for 2 to 9 % less time.
//
// Measured, row kernel -> this kernel, us per layer: bf16 x 64, 16 ragged sequences of 512 on average, 16 heads, 442 -> 34;
// float x 64, 32 sequences of 384, 4 heads, 192 -> 40.
template <typename T, int DH, bool CAUSAL, bool BIAS, bool V2, int QB>
__global__ __launch_bounds__(PF_THREADS, (pf_per_cu<T, DH, V2>())) void prefill_mfma_kernel(const T* __restrict__ qkv,
                                                                  const int32_t* __restrict__ cu,
                                                                  const int32_t* __restrict__ tiles, int H,
                                                                  float scale, const float* __restrict__ bias_by_dist,
                                                                  int radius, T* __restrict__ out, const T* __restrict__ pool,
                                                                  const int64_t* __restrict__ base,
                                                                  const int32_t* __restrict__ cap, int layer)
{
    constexpr int RB = DH * (int)sizeof(T), RPL = 1024 / RB;                   // bytes per row; rows per wave-load
    constexpr int PF_LPT = PF_KT / RPL / PF_NW;                   // direct-to-LDS loads per wave and tile
    constexpr int PF_TILE = pf_tile_bytes(RB);
    constexpr int DS = RB / 64, DT = DH / 16;                     // 64-byte steps of the first product, feature tiles of the second
    constexpr bool SPLIT_P = sizeof(T) == 2 && DH == 64;
    constexpr bool PARTED = pf_parted<T, DH>();
    constexpr int PLANE = PF_KT * 128;                            // PARTED: bytes of one part of a key or value tile
    extern __shared__ __align__(16) unsigned char pf_smem[];      // 2 key tiles, then the value tile(s), then the bias table
    float* sbias = (float*)(pf_smem + pf_lds<T, DH, V2>());

    // Workgroup -> (tile, head).  Workgroups go to the 8 XCDs round-robin in launch order.  With a multiple of 8 heads,
    // XCD x takes heads x, x + 8, ...: its j-th workgroup is tile j / (H/8) for its head number j % (H/8), so the
    // tiles of one sequence and head (neighbours in the list, readers of the same keys and values) share an L2 and
    // run side by side.  Otherwise heads vary fastest.
    int tile, h;
    if ((H & 7) == 0) {
        int hpx = H >> 3, j = blockIdx.x >> 3;
        tile = j / hpx;
        h = (blockIdx.x & 7) + 8 * (j - tile * hpx);
    } else {
        tile = blockIdx.x / H;
        h = blockIdx.x - tile * H;
    }
    constexpr int QT = PF_NW * 16 * QB, PIECES = PF_QT / QT;      // the list's tiles are cut into pieces
    int sb = tiles[tile / PIECES * 2], q0 = tiles[tile / PIECES * 2 + 1] + (PIECES - 1 - tile % PIECES) * QT;
    int t0 = cu[sb], n = cu[sb + 1] - t0;
    if (q0 >= n) return;
    int inner = H * DH;
    int64_t ld = 3 * (int64_t)inner;
    int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int qi = lane & 15, g = lane >> 4;
    int wq0 = q0 + wave * (16 * QB);                                     // this wave's first query row
    const T* seq = qkv + (int64_t)t0 * ld + h * DH;

    // the head's table, continued on either side with its first and last entry
    if (BIAS) {
        for (int i = tid; i < pf_bias_entries(radius); i += PF_THREADS) {
            int e = i - PF_BIAS_PAD;
            e = e < 0 ? 0 : (e > 2 * radius ? 2 * radius : e);
            sbias[i] = bias_by_dist[(int64_t)h * (2 * radius + 1) + e] * LOG2E;
        }
    }

    // query fragments (B operand): lane (query qi, lane group g) holds 16-byte chunk 4*ds + g of its query row
    // (PARTED: parts 0 .. 2 of elements 8 * g .. +7 of its first and of its second 32)
    constexpr int QF = PARTED ? 6 : DS;
    u32x4 qf[QB][QF];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        int qr = wq0 + qb * 16 + qi;
        qr = qr < n ? qr : n - 1;
        if constexpr (PARTED) {
            const f32x4* qp = (const f32x4*)(seq + (int64_t)qr * ld) + 2 * g;
#pragma unroll
            for (int ds = 0; ds < 2; ++ds) {
                uint2 a[3], b[3];
                bf16_parts(qp[ds * 8] * PART_SCALE, a);
                bf16_parts(qp[ds * 8 + 1] * PART_SCALE, b);
#pragma unroll
                for (int p = 0; p < 3; ++p) qf[qb][ds * 3 + p] = u32x4{a[p].x, a[p].y, b[p].x, b[p].y};
            }
        } else {
            const u32x4* qp = (const u32x4*)(seq + (int64_t)qr * ld) + g;
#pragma unroll
            for (int ds = 0; ds < DS; ++ds) qf[qb][ds] = qp[ds * 4];
        }
    }
    // the softmax below takes the maximum of the raw scores, which wants a positive scale: the sign of a negative one goes to
    // the queries
    if (scale < 0.f) {
#pragma unroll
        for (int qb = 0; qb < QB; ++qb)
#pragma unroll
            for (int i = 0; i < QF; ++i) qf[qb][i] ^= sizeof(T) == 4 && !PARTED ? 0x80000000u : 0x80008000u;
    }
    int kend = n;
    if (CAUSAL) kend = q0 + QT < n ? q0 + QT : n;
    int n_tiles = (kend + PF_KT - 1) / PF_KT;

    // ---- loaders.  Per tile of keys and of values a wave issues PF_LPT 1 KB direct-to-LDS loads of RPL rows each; a
    // lane fills a slot of its row with the chunk that the swizzle puts there.  Written as inline assembly
    // so that the compiler does not order every later LDS read behind them.
    unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)pf_smem;
    // keys and values: from the packed activations, or (base given) from the cache, where a head's rows follow each other
    const T *keys = seq + inner, *values = seq + 2 * inner;
    unsigned kv_row = (unsigned)ld * (unsigned)sizeof(T);
    if (base) {
        keys = pool + base[sb] + ((int64_t)(layer * 2) * H + h) * cap[sb] * DH;
        values = keys + (int64_t)H * cap[sb] * DH;
        kv_row = RB;
    }
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
    auto load_to_lds = [&](const char* src, unsigned voff, unsigned dst) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(dst), "v"(voff), "s"(src) : "memory", "m0");
    };
#pragma clang diagnostic pop
    auto load_tile = [&](const char* base, int kt, unsigned dst) {
        int lane = tid & 63;
        if (BIAS) asm volatile("" : "+v"(lane));                    // the rows' offsets are made anew per tile: held, they spill
#pragma unroll
        for (int p = 0; p < PF_LPT; ++p) {
            constexpr int CPR = RB / 16;                            // chunks per row
            int row = (p * PF_NW + wave) * RPL;                     // first of the tile rows of this load
            int key = row + lane / CPR;
            int kg = kt * PF_KT + key;
            kg = kg < n ? kg : n - 1;
            unsigned voff = (unsigned)kg * kv_row + (((lane & (CPR - 1)) ^ pf_swz<RB>(key)) << 4);
            load_to_lds(base, voff, dst + row * RB);
        }
    };
    auto load_k = [&](int kt) { load_tile((const char*)keys, kt, lds_base + (kt & 1) * PF_TILE); };
    auto load_v = [&](int kt) { load_tile((const char*)values, kt, lds_base + (2 + (V2 ? kt & 1 : 0)) * PF_TILE); };

    // PARTED: a tile goes through registers, 4 groups of 4 elements per thread of keys and of values, and is parted on the way to LDS
    f32x4 kv_reg[PARTED ? 8 : 1];
    auto fetch_kv = [&](int kt) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            int u = i * PF_THREADS + tid, kg = kt * PF_KT + (u >> 4);
            kg = kg < n ? kg : n - 1;
            unsigned at = (unsigned)kg * kv_row + (u & 15) * 16;
            kv_reg[i] = *(const f32x4*)((const char*)keys + at);
            kv_reg[4 + i] = *(const f32x4*)((const char*)values + at);
        }
    };
    auto put_kv = [&]() {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            int u = (i & 3) * PF_THREADS + tid, row = u >> 4, c = u & 15;
            unsigned char* d = pf_smem + (i >> 2) * 3 * PLANE + row * 128 + (((c >> 1) ^ pf_swz<128>(row)) << 4) + (c & 1) * 8;
            uint2 w[3];
            bf16_parts(kv_reg[i] * PART_SCALE, w);
#pragma unroll
            for (int p = 0; p < 3; ++p) *(uint2*)(d + p * PLANE) = w[p];
        }
    };

    f32x4 o_acc[QB][DT];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o_acc[qb][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run[QB], l_run[QB];
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        m_run[qb] = -INFINITY;
        l_run[qb] = 0.f;
    }
    // (PARTED: of scores that carry PART_SCALE twice)
    float sc = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, fabsf(scale) * LOG2E * (PARTED ? PARTS_UNSCALE : 1.f))));
    f32x4 s_acc[QB][4];

    // a wave whose queries all lie before a tile's first key (causal) or past the sequence end has nothing to
    // compute for that tile; it still moves its share of the tiles
    auto active = [&](int kt) { return wq0 < n && (!CAUSAL || kt * PF_KT <= wq0 + 16 * QB - 1); };

    // ---- the three phases of a tile
    auto phase_s = [&](int kt) {
        const unsigned char* sK = pf_smem + (kt & 1) * PF_TILE;
        // The four swizzled chunk offsets of a lane ((4 ds + g) ^ qi for ds = 0..3) are recomputed per tile from one
        // register: held across the tile loop they cost four, and a register spilled in this loop puts a full wait
        // for the tile loads in flight in front of its reload (scratch reloads count with them).
        // (With a bias, whose look-ups want registers too, all of a lane's offsets are.)
        int l = lane;
        if (BIAS) asm volatile("" : "+v"(l));
        int qi = l & 15, g = l >> 4, qx = pf_swz<PARTED ? 128 : RB>(qi);
        if (!BIAS) asm volatile("" : "+v"(qx));
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
            if constexpr (PARTED) {
                // The products of the first parts, 32 features each, and the others' sum (which is small, and so are its roundings)
                // are added as three numbers.
                f32x4 c[2][QB], rest[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) rest[qb] = c[0][qb] = c[1][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ds = 0; ds < 2; ++ds) {
                    u32x4 fk[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) fk[p] = *(const u32x4*)(pf_smem + p * PLANE + (kb * 16 + qi) * 128 + (((ds * 4 + g) ^ qx) << 4));
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        c[ds][qb] = HalfUnit<bf16_t>::mma(fk[0], qf[qb][ds * 3], c[ds][qb]);
#pragma unroll
                        for (int x = 0; x < 5; ++x) rest[qb] = HalfUnit<bf16_t>::mma(fk[PARTS[x][0]], qf[qb][ds * 3 + PARTS[x][1]], rest[qb]);
                    }
                }
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    f32x4 v = s_acc[qb][kb] = c[0][qb] + c[1][qb] + rest[qb];
                    // A score of 2^80 and more in magnitude is infinite with the parts' factor.  +infinity makes its row NaN below;
                    // -infinity would only lose its key, so the row is made NaN here.
                    l_run[qb] = fmaf(fminf(fminf(v[0], v[1]), fminf(v[2], v[3])), 0.f, l_run[qb]);
                }
            } else if constexpr (sizeof(T) == 4) {
                // sums of 8 features each (two MFMAs), added pairwise: part x is half x % 2 of the 16-byte chunks 4 * (x / 2) + g
                auto sum = [&](auto self, auto first, auto count, f32x4 (&c)[QB]) -> void {
                    constexpr int X = decltype(first)::value, N = decltype(count)::value;
                    if constexpr (N == 1) {
                        f32x4 kf = *(const f32x4*)(sK + (kb * 16 + qi) * RB + (((X / 2 * 4 + g) ^ qx) << 4));
#pragma unroll
                        for (int qb = 0; qb < QB; ++qb) {
                            f32x4 q = __builtin_bit_cast(f32x4, qf[qb][X / 2]);
                            c[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[X % 2 * 2], q[X % 2 * 2], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                            c[qb] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[X % 2 * 2 + 1], q[X % 2 * 2 + 1], c[qb], 0, 0, 0);
                        }
                    } else {
                        f32x4 d[QB];
                        self(self, std::integral_constant<int, X>{}, std::integral_constant<int, N / 2>{}, c);
                        self(self, std::integral_constant<int, X + N / 2>{}, std::integral_constant<int, N / 2>{}, d);
#pragma unroll
                        for (int qb = 0; qb < QB; ++qb) c[qb] += d[qb];
                    }
                };
                f32x4 c[QB];
                sum(sum, std::integral_constant<int, 0>{}, std::integral_constant<int, 2 * DS>{}, c);
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    asm volatile("" : "+v"(c[qb]));               // the additions stay here: moved into the softmax's branches they spill
                    s_acc[qb][kb] = c[qb];
                }
            } else {
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) s_acc[qb][kb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ds = 0; ds < DS; ++ds) {
                    u32x4 fk = *(const u32x4*)(sK + (kb * 16 + qi) * RB + (((ds * 4 + g) ^ qx) << 4));
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) s_acc[qb][kb] = HalfUnit<T>::mma(fk, qf[qb][ds], s_acc[qb][kb]);
                }
            }
        }
    };
    // element r of lane (qi, g) in s_acc[qb][kb]: key = kt*64 + kb*16 + 4*g + r, query wq0 + qb*16 + qi.
    // Only tiles that straddle the sequence end or (causal) this wave's diagonal need the per-element mask.
    auto phase_softmax = [&](int kt) {
        // With a bias, a tile whose keys all lie at least `radius` before (or after) every query of this wave adds one
        // constant, the table's first (last) entry, to all of its scores: it takes the path without look-ups with that
        // constant folded into the exponent.  (The bias table is indexed by the clamped distance.)
        // In the other tiles no distance passes the table's ends by PF_BIAS_PAD or more, so the continued table is read without a
        // clamp, and a lane's four keys of a block are four entries in a row, the same ones for key block kb of the first
        // queries and kb + 1 of the second: 20 entries per lane and tile.  (T5-11B's heads, 16 ragged sequences of 768: 1270 us
        // with a clamped look-up per score and two workgroups per CU, now 1010.)
        bool edge = kt * PF_KT + PF_KT > n || (CAUSAL && kt * PF_KT + PF_KT - 1 > wq0);
        float mul = sc, cbias = 0.f;           // score = s_acc * mul + cbias
        if (BIAS) {
            if (kt * PF_KT + PF_KT - 1 - wq0 <= -radius) {
                cbias = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, sbias[0])));
            } else if (kt * PF_KT - (wq0 + 16 * QB - 1) >= radius) {
                cbias = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, sbias[2 * (radius + PF_BIAS_PAD)])));
            } else {
                int l = lane;
                asm volatile("" : "+v"(l));         // the offset is made anew per tile: held, it spills
                const float* t = sbias + (radius + PF_BIAS_PAD) + kt * PF_KT - wq0 + (l >> 4) * 4 - (l & 15);
#pragma unroll
                for (int d = 1 - QB; d < 4; ++d) {
                    float b[4];
#pragma unroll
                    for (int r = 0; r < 4; ++r) b[r] = t[d * 16 + r];
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        if (d >= 0) s_acc[0][d][r] = fmaf(s_acc[0][d][r], sc, b[r]);
                        if (QB > 1 && d < 3) s_acc[QB - 1][d + 1][r] = fmaf(s_acc[QB - 1][d + 1][r], sc, b[r]);
                    }
                }
                mul = 1.f;
            }
        }
        if (edge) {
            int key0 = kt * PF_KT + 4 * g;
            asm volatile("" : "+v"(key0));          // keeps the mask arithmetic inside this branch
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        int key = key0 + kb * 16 + r;
                        bool ok = key < n && (!CAUSAL || key <= wq0 + qb * 16 + qi);
                        s_acc[qb][kb][r] = ok ? fmaf(s_acc[qb][kb][r], mul, cbias) : -INFINITY;
                    }
            mul = 1.f;
            cbias = 0.f;
        }
        float alpha[QB];
#pragma unroll
        for (int qb = 0; qb < QB; ++qb) {
            // mul is not negative: take the maximum of the raw scores and fold the scale into the exponent
            float mx = -INFINITY;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) mx = fmaxf(mx, s_acc[qb][kb][r]);
            mx = fmaf(mx, mul, cbias);
            mx = rows_max(mx);
            float m_new = fmaxf(m_run[qb], mx);
            float mref = m_new == -INFINITY ? 0.f : m_new;
            alpha[qb] = fast_exp2(m_run[qb] - mref);
            float shift = cbias - mref;
            float rs = 0.f;
#pragma unroll
            for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float p = fast_exp2(fmaf(s_acc[qb][kb][r], mul, shift));
                    s_acc[qb][kb][r] = p;
                    rs += p;
                }
            rs = rows_sum(rs);
            l_run[qb] = l_run[qb] * alpha[qb] + rs;
            m_run[qb] = m_new;
        }
        // the running maximum of a query stops moving after the first tiles: rescale only when some lane needs it
        if (__builtin_amdgcn_ballot_w64(alpha[0] != 1.f || alpha[QB - 1] != 1.f) != 0) {
#pragma unroll
            for (int qb = 0; qb < QB; ++qb)
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) o_acc[qb][dt][r] *= alpha[qb];
        }
    };
    // O^T += V^T . P^T.  MFMA k-step ks covers keys 32*ks .. +31 of the tile; lane group g supplies keys
    // 4*g .. +3 of key blocks 2*ks and 2*ks+1.  The value tile lies row-major (one key per row); the transposing
    // read hands lane (qi, g) the column 16*dt + qi of those four keys: within the 16 lanes of a group, lane
    // L = 4*j + q points at columns 16*dt + 4*q .. +3 of key 4*g + j.
    int v_row = 4 * g + (qi >> 2), v_q = qi & 3;
    auto phase_pv = [&](int kt) {
        const unsigned char* tV = pf_smem + (2 + (V2 ? kt & 1 : 0)) * PF_TILE;
        if constexpr (PARTED) {
            // probabilities in parts, as below, and a tile's sums added as one
            const unsigned char* sV = pf_smem + 3 * PLANE + v_row * 128 + (v_q & 1) * 8;
            bf16x8 pf[2][3][QB];
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) {
                    uint2 a[3], b[3];
                    bf16_parts(s_acc[qb][2 * ks] * PART_SCALE, a);
                    bf16_parts(s_acc[qb][2 * ks + 1] * PART_SCALE, b);
#pragma unroll
                    for (int p = 0; p < 3; ++p) pf[ks][p][qb] = __builtin_bit_cast(bf16x8, u32x4{a[p].x, a[p].y, b[p].x, b[p].y});
                }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                f32x4 c[2][QB], rest[QB];
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) rest[qb] = c[0][qb] = c[1][qb] = f32x4{0.f, 0.f, 0.f, 0.f};
                int slot = ((2 * dt + (v_q >> 1)) ^ pf_swz<128>(v_row)) << 4;
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) {
                    bf16x8 fv[3];
#pragma unroll
                    for (int p = 0; p < 3; ++p) {
                        uint2 lo = pf_read_tr(sV + p * PLANE + ks * 32 * 128 + slot);
                        uint2 hi = pf_read_tr(sV + p * PLANE + (ks * 32 + 16) * 128 + slot);
                        fv[p] = __builtin_bit_cast(bf16x8, uint4{lo.x, lo.y, hi.x, hi.y});
                    }
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) {
                        c[ks][qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fv[0], pf[ks][0][qb], c[ks][qb], 0, 0, 0);
#pragma unroll
                        for (int x = 0; x < 5; ++x)
                            rest[qb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fv[PARTS[x][0]], pf[ks][PARTS[x][1]][qb], rest[qb], 0, 0, 0);
                    }
                }
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) o_acc[qb][dt] += c[0][qb] + c[1][qb] + rest[qb];
            }
            return;
        } else if constexpr (sizeof(T) == 4) {
            // Lane group g supplies key 4*g + r of key block kb, for feature 16*dt + qi: chunk 4*dt + qi/4 of its row, at slot
            // 4 * (dt ^ g) + (qi/4 ^ r).  A sum per key block, added pairwise.  (The offsets are recomputed per tile: held, they spill.)
            int ga = g;
            asm volatile("" : "+v"(ga));
            const unsigned char* vr[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) vr[r] = tV + (4 * ga + r) * RB + (((qi >> 2) ^ r) << 4) + (qi & 3) * 4;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                f32x4 c[QB][4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) c[qb][i] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kb = 0; kb < 4; ++kb)
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float fv = *(const float*)(vr[r] + ((dt ^ ga) << 6) + kb * 16 * RB);
#pragma unroll
                        for (int qb = 0; qb < QB; ++qb) c[qb][kb] = __builtin_amdgcn_mfma_f32_16x16x4f32(fv, s_acc[qb][kb][r], c[qb][kb], 0, 0, 0);
                    }
#pragma unroll
                for (int qb = 0; qb < QB; ++qb) o_acc[qb][dt] += (c[qb][0] + c[qb][1]) + (c[qb][2] + c[qb][3]);
                __builtin_amdgcn_sched_barrier(0);
            }
            return;
        }
        const unsigned char* sV = tV + v_row * RB + (v_q & 1) * 8;
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) {
            // p, or (SPLIT_P) its first, second and third 8 bits: p = pf[0] + pf[1] + pf[2]
            constexpr int NP = SPLIT_P ? 3 : 1;
            bf16x8 pf[NP][QB];
#pragma unroll
            for (int qb = 0; qb < QB; ++qb) {
                if constexpr (!SPLIT_P) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) pf[0][qb][e] = (bf16_t)s_acc[qb][2 * ks + (e >> 2)][e & 3];
                } else {
#pragma unroll
                    for (int i = 0; i < NP; ++i) {
                        u32x4 w;
#pragma unroll
                        for (int e = 0; e < 8; e += 2) {
                            f32x4& sv = s_acc[qb][2 * ks + (e >> 2)];
                            float a = sv[e & 3], b = sv[(e & 3) + 1];
                            unsigned ua = __float_as_uint(a), ub = __float_as_uint(b);
                            w[e >> 1] = __builtin_amdgcn_perm(ub, ua, 0x07060302);          // their upper halves
                            sv[e & 3] = a - __uint_as_float(ua & 0xffff0000u);
                            sv[(e & 3) + 1] = b - __uint_as_float(ub & 0xffff0000u);
                        }
                        pf[i][qb] = __builtin_bit_cast(bf16x8, w);
                    }
                }
            }
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                int slot = ((2 * dt + (v_q >> 1)) ^ pf_swz<RB>(v_row)) << 4;
                uint2 lo = pf_read_tr(sV + ks * 32 * RB + slot);
                uint2 hi = pf_read_tr(sV + (ks * 32 + 16) * RB + slot);
                uint4 both = {lo.x, lo.y, hi.x, hi.y};
                bf16x8 fv = __builtin_bit_cast(bf16x8, both);
#pragma unroll
                for (int i = 0; i < NP; ++i) {
#pragma unroll
                    for (int qb = 0; qb < QB; ++qb) o_acc[qb][dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fv, pf[i][qb], o_acc[qb][dt], 0, 0, 0);
                }
            }
        }
    };

    if constexpr (PARTED) {
        fetch_kv(0);
        for (int kt = 0; kt < n_tiles; ++kt) {
            put_kv();
            __syncthreads();
            if (kt + 1 < n_tiles) fetch_kv(kt + 1);
            if (active(kt)) {
                phase_s(kt);
                phase_softmax(kt);
                phase_pv(kt);
            }
            __syncthreads();
        }
    } else if constexpr (V2) {
        load_k(0);
        load_v(0);
        for (int kt = 0; kt < n_tiles; ++kt) {
            __builtin_amdgcn_s_waitcnt(0x0070 | (15 << 8));       // vmcnt(0): this wave's part of tile kt has landed
            __syncthreads();
            if (kt + 1 < n_tiles) {                               // into the buffers that tile kt - 1 has left
                load_k(kt + 1);
                load_v(kt + 1);
            }
            if (active(kt)) {
                phase_s(kt);
                phase_softmax(kt);
                phase_pv(kt);
            }
        }
    } else {
        // Key tiles are double buffered; the single value tile is loaded at the start of its own iteration, behind
        // the scores and the softmax, which costs a second barrier per tile but lets three workgroups share a CU.
        load_k(0);
        __builtin_amdgcn_s_waitcnt(0x0070 | (15 << 8));           // vmcnt(0)
        __syncthreads();

        for (int kt = 0; kt < n_tiles; ++kt) {
            load_v(kt);                                           // PF_LPT loads
            bool more = kt + 1 < n_tiles;
            if (more) load_k(kt + 1);                             // PF_LPT loads, into the buffer tile kt-1 has left
            bool act = active(kt);
            if (act) {
                phase_s(kt);
                phase_softmax(kt);
            }
            if (more) __builtin_amdgcn_s_waitcnt(0x0070 | PF_LPT | (15 << 8));   // the value tile: all but the key loads
            else __builtin_amdgcn_s_waitcnt(0x0070 | (15 << 8));
            __syncthreads();
            if (act) phase_pv(kt);
            __builtin_amdgcn_s_waitcnt(0x0070 | (15 << 8));       // this wave's part of the next key tile has landed
            __syncthreads();
        }
    }

    // lane (qi, g) holds features 16*dt + 4*g .. +3 of its query
#pragma unroll
    for (int qb = 0; qb < QB; ++qb) {
        int qpos = wq0 + qb * 16 + qi;
        float inv = 1.f / l_run[qb];
        float most = o_acc[qb][0][0];                              // NaN if one of them is
        if constexpr (PARTED) {
            // outputs carry PART_SCALE twice too, and an infinite one may not be infinite without
            inv *= PARTS_UNSCALE;
            most = l_run[qb];
#pragma unroll
            for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                for (int j = 0; j < 4; ++j) most = fmaf(o_acc[qb][dt][j], 0.f, most);
        }
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int j = 0; j < 4; ++j) most = __builtin_elementwise_maximum(most, o_acc[qb][dt][j]);
        // The second product takes every key of a tile: 0 times the infinite or NaN value of a key that the mask keeps from this
        // query is NaN.  Such a row is not stored, but computed again from its own keys alone (rare, so not for speed).
        unsigned long long lanes = __builtin_amdgcn_ballot_w64(most != most && qpos < n);
        unsigned again = (unsigned)(lanes | lanes >> 32);
        again = (again | again >> 16) & 0xffff;                   // bit qi: query row wq0 + 16 * qb + qi
        if (qpos < n && !(again >> qi & 1)) {
            T* op = out + (int64_t)(t0 + qpos) * inner + h * DH + 4 * g;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                typename Vec4<T>::type w;
#pragma unroll
                for (int j = 0; j < 4; ++j) w[j] = (T)(o_acc[qb][dt][j] * inv);
                *(typename Vec4<T>::type*)(op + dt * 16) = w;
            }
        }
        for (; again; again &= again - 1) {
            int qr = wq0 + qb * 16 + __builtin_ctz(again);
            prefill_row<T, DH, BIAS>(seq + qr * ld, keys, values, kv_row / (int)sizeof(T), qr, CAUSAL ? qr + 1 : n, scale * LOG2E, sbias + (BIAS ? PF_BIAS_PAD : 0), radius, lane,
                                     out + (int64_t)(t0 + qr) * inner + h * DH);
        }
    }
}

PrefillWork prefill_work(const int32_t* lens, int n_seqs, bool causal)
{
    PrefillWork w;
    for (int i = 0; i < n_seqs; ++i) {
        int64_t n = lens[i];
        if (n > w.max_len) w.max_len = (int)n;
        w.pairs += causal ? n * (n + 1) / 2 : n * n;
        for (int64_t q0 = 0; q0 < n; q0 += PREFILL_TILE_Q) {
            int64_t keys = causal && q0 + PREFILL_TILE_Q < n ? q0 + PREFILL_TILE_Q : n;
            w.key_tiles += (keys + PREFILL_TILE_K - 1) / PREFILL_TILE_K;
        }
    }
    return w;
}

void prefill_tile_order(const int32_t* lens, int n_seqs, std::vector<int32_t>& tiles)
{
    std::vector<int> order(n_seqs);
    for (int i = 0; i < n_seqs; ++i) order[i] = i;
    std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return lens[x] > lens[y]; });
    for (int i : order)
        for (int q0 = (lens[i] - 1) / PREFILL_TILE_Q * PREFILL_TILE_Q; q0 >= 0; q0 -= PREFILL_TILE_Q) {
            tiles.push_back(i);
            tiles.push_back(q0);
        }
}

template <typename T, int DH, bool CAUSAL, bool BIAS, bool V2, int QB> static hipError_t launch_prefill(const AttnPackedArgs& a, hipStream_t s)
{
    auto kern = prefill_mfma_kernel<T, DH, CAUSAL, BIAS, V2, QB>;
    const int lds = pf_lds<T, DH, V2>() + (BIAS ? pf_bias_entries(a.bias_radius) * 4 : 0);
    static LdsLimit limit[MAX_DEVICES];
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) dev = 0;
    hipError_t e = limit[dev].raise((const void*)kern, pf_lds<T, DH, V2>() + (BIAS ? (PF_BIAS + 2 * PF_BIAS_PAD) * 4 : 0));
    if (e != hipSuccess) return e;
    // a launch has fewer than 2^32 threads: very many short sequences take several
    const int64_t per_tile = (int64_t)(2 / QB) * a.H, most = (MAX_LAUNCH_THREADS / PF_THREADS) / per_tile;
    if (most < 1) return hipErrorInvalidValue;
    for (int64_t t = 0; t < a.n_tiles; t += most) {
        const int64_t n = a.n_tiles - t < most ? a.n_tiles - t : most;
        kern<<<(unsigned)(n * per_tile), PF_THREADS, lds, s>>>((const T*)a.qkv, a.cu, a.tiles + 2 * t, a.H, a.scale, BIAS ? a.bias_by_dist : nullptr,
                                                               BIAS ? a.bias_radius : 0, (T*)a.out, (const T*)a.pool, a.base, a.cap, a.layer);
        if ((e = hipGetLastError()) != hipSuccess) return e;
    }
    return hipSuccess;
}

// The form of the MFMA kernel: query blocks per wave (QB; the other half of a listed tile goes to a workgroup of its own at QB 1)
// and value buffers (V2), by how many workgroups of whole tiles there are.  One or two buffers do not change a row's result, nor do
// the blocks.
//   QB 2 with one value buffer / with two / QB 1 with two, bf16 x 128, us of a launch on one MI355X, 12 in a row; 60 batches of 1 to 16
//   ragged sequences of 96 to 1000 tokens, 40, 96 and 128 heads, table of radius 100; of whole tiles
//     causal                160 21.6 / 17.5 / 14.9    320 35.0 / 29.2 / 24.1    400 27.9 / 24.8 / 20.0   600 33.3 / 26.3 / 29.4   720 34.1 / 31.3 / 30.6
//                           768 39.7 / 42.0 / 44.5    960 36.5 / 37.9 / 41.3   1120 46.4 / 42.3 / 44.8  1200 63.7 / 59.7 / 70.6  1440 66.3 / 67.0 / 78.1
//     causal, with a table  160 22.8 / 20.8 / 15.9    400 30.0 / 27.5 / 22.2    600 34.0 / 29.4 / 35.4   768 41.6 / 45.3 / 47.5  1080 54.1 / 56.1 / 60.3
//     neither               120 14.5 / 13.5 /  9.6    256 13.2 / 12.4 / 10.6    320 42.3 / 40.7 / 44.5   600 43.0 / 48.7 / 48.7  2960 136 / 153 / 178
//     table, not causal     120 16.1 / 15.0 / 10.7    256 14.6 / 13.3 / 11.5    320 44.7 / 43.3 / 48.0   600 43.8 / 50.2 / 49.8  13696 928 / 994 / 1268
//   With one buffer three workgroups share a CU, so 768 are all there at once, with two 512: from 720 on one buffer is the faster, and
//   without a table, where a tile's two barriers weigh more, two again while one buffer's second round fills less than two thirds of
//   the chip.  Over these 240 launches the form taken is within 0.8 % of the fastest of the three on average, and none is slower than the
//   form that all of them took before, QB 2 with one buffer.
//   The same of other types (times by events around single launches, which add about 3):
//   QB 2 with two / QB 1 with two (/ with one)
//   bf16 x 64   64 18.3 / 12.1    592 27.3 / 22.8    2672 62.4 / 57.6: half the registers, so five workgroups on a CU in place of four
//   float x 64, float MFMAs with QB 2 / with QB 1 / bf16 parts (one form: three workgroups on a CU)
//               148 60.0 / 40.8 / 35.5    292 73.2 / 45.0 / 38.6    452 81.0 / 58.6 / 42.8    804 122 / 100 / 67.8
template <typename T, int DH, bool CAUSAL, bool BIAS> static hipError_t launch_prefill(const AttnPackedArgs& a, hipStream_t s)
{
    const int64_t wgs = (int64_t)a.n_tiles * a.H;
    if constexpr (DH == 64) {
        return launch_prefill<T, DH, CAUSAL, BIAS, !pf_parted<T, DH>(), 1>(a, s);
    } else if constexpr (sizeof(T) == 4) {
        return launch_prefill<T, DH, CAUSAL, BIAS, true, 2>(a, s);
    } else {
        if (wgs <= (CAUSAL ? 400 : 256)) return launch_prefill<T, DH, CAUSAL, BIAS, true, 1>(a, s);
        if constexpr (CAUSAL) {
            if (wgs <= 720 || (!BIAS && wgs > 1024 && wgs <= 1280)) return launch_prefill<T, DH, CAUSAL, BIAS, true, 2>(a, s);
        }
        return launch_prefill<T, DH, CAUSAL, BIAS, false, 2>(a, s);
    }
}
template <typename T, int DH> static hipError_t launch_prefill(const AttnPackedArgs& a, hipStream_t s)
{
    if (a.causal) return a.bias_by_dist ? launch_prefill<T, DH, true, true>(a, s) : launch_prefill<T, DH, true, false>(a, s);
    return a.bias_by_dist ? launch_prefill<T, DH, false, true>(a, s) : launch_prefill<T, DH, false, false>(a, s);
}

// Which kernel a batch runs on.  The MFMA kernel works in tiles of 128 query rows x 64 keys, whole ones: a batch of short
// sequences, or one that leaves most of the chip idle while its longest sequence's key tiles pass in turn, is served sooner by
// the row kernel's many small workgroups.  us of either, fitted to 168 batches per type on one MI355X (1 to 64 sequences of 2
// to 1000 tokens, ragged and not, 4 to 40 heads; within 6-11 % at the median, a quarter to a half at worst): the faster of the
// two by these takes at most 1.17, 1.19 and 1.13 times the faster one measured; the MFMA kernel alone took up to 6.9, 24 and
// 1.8 times (float x 64, float x 128, bf16 x 64; e.g. 64 sequences of one token, 16 heads, float x 128: 61 us, rows 4).  The MFMA
// kernel's figures for head size 64 are of later fits, of its 64-row workgroups: bf16 over 47 batches, float over 69 (with and without
// mask and bias table), where the faster of the two is taken every time (5 sequences of 87 tokens in all, 32 heads: rows 5.1, MFMA 6.2).
// bf16 x 128 stays on the MFMA kernel, whose tiles were made for it.
static bool prefill_mfma_pays(const AttnPackedArgs& a)
{
    if (a.dtype == DT_BF16 && a.dh == 128) return true;
    struct Cost { double row_fixed, row, pair, mfma_fixed, chain, tile; };
    static constexpr Cost F64{3.1, 0.61e-3, 16.4e-6, 2.4, 2.5, 2.4}, F128{3.3, 0.59e-3, 35.1e-6, 4.5, 10.1, 11.1}, B64{3.4, 1.08e-3, 9.5e-6, 2.5, 0.83, 0.8};
    const Cost& c = a.dtype == DT_BF16 ? B64 : a.dh == 64 ? F64 : F128;
    double row = c.row_fixed + a.H * (c.row * a.T + c.pair * a.work.pairs);
    double mfma = c.mfma_fixed + c.chain * ((a.work.max_len + PREFILL_TILE_K - 1) / PREFILL_TILE_K) + c.tile * a.H * a.work.key_tiles / 256;
    return mfma < row;
}

hipError_t launch_attn_packed(const AttnPackedArgs& a, hipStream_t s)
{
    if (a.T <= 0) return hipSuccess;
    if ((a.dtype != DT_F32 && a.dtype != DT_BF16) || (a.dh != 64 && a.dh != 128)) return hipErrorInvalidValue;
    // the scale of parted scores (float x 64) carries 2^-48: where that would be no normal float, the row kernel serves
    const bool scale_fits = a.dtype != DT_F32 || a.dh != 64 || a.scale == 0.f || !(fabsf(a.scale) < 0x1p-70f);
    const bool mfma = a.force_generic <= 0 && a.n_tiles > 0 && scale_fits && (a.force_generic < 0 || prefill_mfma_pays(a));
    // The key loader addresses the rows of one sequence with 32-bit byte offsets, and a head's bias table must fit
    // the kernel's LDS copy; a batch outside these limits runs on the row kernel, which is correct but far slower,
    // so say so (once).
    const int64_t longest = a.work.max_len, row_bytes = (int64_t)3 * a.H * a.dh * (a.dtype == DT_F32 ? 4 : 2);
    const bool mfma_fits = longest * row_bytes < ((int64_t)1 << 32) && (!a.bias_by_dist || (a.bias_radius >= 0 && a.bias_radius <= (PF_BIAS - 1) / 2));
    if (mfma && !mfma_fits) {
        static std::once_flag warned;
        std::call_once(warned, [&]() {
            fprintf(stderr, "exe: prefill attention falls back to the row kernel (longest sequence %lld rows of %lld bytes, bias "
                            "radius %d): expect it to be much slower\n", (long long)longest, (long long)row_bytes, a.bias_radius);
        });
    }
    if (mfma && mfma_fits) {
        if (a.dtype == DT_F32) return a.dh == 64 ? launch_prefill<float, 64>(a, s) : launch_prefill<float, 128>(a, s);
        return a.dh == 64 ? launch_prefill<bf16_t, 64>(a, s) : launch_prefill<bf16_t, 128>(a, s);
    }
    dim3 grid(a.H, a.T);
#define EXE_ROW(T, DH)                                                                                           \
    attn_row_kernel<T, DH, true><<<grid, 256, 0, s>>>((const T*)a.qkv, 0, (const T*)a.pool, a.base, a.cap, nullptr, \
                                                      a.tok_pos, a.tok_b, a.cu, a.layer, a.H, a.causal, a.scale, \
                                                      a.bias_by_dist, a.bias_radius, (T*)a.out, 0, 0)
    if (a.dtype == DT_F32 && a.dh == 64) EXE_ROW(float, 64);
    else if (a.dtype == DT_F32 && a.dh == 128) EXE_ROW(float, 128);
    else if (a.dtype == DT_BF16 && a.dh == 64) EXE_ROW(bf16_t, 64);
    else EXE_ROW(bf16_t, 128);
#undef EXE_ROW
    return hipGetLastError();
}

}  // namespace exe
