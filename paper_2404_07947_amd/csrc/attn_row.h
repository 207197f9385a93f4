// One query row against keys and values of one head, by one workgroup: what the row kernel (kernels_attn.hip) and the fused
// decode block of small models (kernels_small.hip) share.
#pragma once
#include <type_traits>

#include "common.h"

namespace exe {

constexpr float LOG2E = 1.44269504088896340736f;
constexpr int ATTN_BIAS_LDS = 1024;       // entries of a head's bias table that the row kernel keeps in LDS

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// the value of the lane `lane ^ O`
template <int O> __device__ __forceinline__ float lane_xor(float x)
{
    if (O == 8) return dpp_move<0x128>(x);   // row_ror:8
    return __shfl_xor(x, O, WAVE);
}

template <typename T, int EPL> struct Chunk;
template <> struct Chunk<float, 4> {
    static __device__ __forceinline__ void unpack(uint4 u, float* f)
    {
        f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y); f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
    }
};
template <> struct Chunk<bf16_t, 8> {
    static __device__ __forceinline__ void unpack(uint4 u, float* f)
    {
        f[0] = bf16lo(u.x); f[1] = bf16hi(u.x); f[2] = bf16lo(u.y); f[3] = bf16hi(u.y);
        f[4] = bf16lo(u.z); f[5] = bf16hi(u.z); f[6] = bf16lo(u.w); f[7] = bf16hi(u.w);
    }
};

// 16 bytes from global memory.  STREAM marks data that is read once (a sequence's cached keys and values during
// decode): a nontemporal load keeps it from displacing other lines in L2, measured 6.3 -> 6.9 .. 7.1 TB/s.
template <bool STREAM, typename T> __device__ __forceinline__ uint4 load_chunk(const T* p)
{
    if (STREAM) {
        typedef unsigned v4u_t __attribute__((ext_vector_type(4)));
        v4u_t t = __builtin_nontemporal_load((const v4u_t*)p);
        return uint4{t.x, t.y, t.z, t.w};
    }
    return *(const uint4*)p;
}

// Paged cache indexing, shared by the kernel and by the host-side check paged_index_check below.
// paged_lookup_row: the row whose block look-up x of the step starting at row j names (nc rows are cached);
// paged_lane_row: the row that the lane group rg of load u of that step reads.
__host__ __device__ __forceinline__ int paged_lookup_row(int j, int x, int rpw, int nc)
{
    int row = j + x * rpw;
    return row < nc ? row : nc - 1;
}
__host__ __device__ __forceinline__ int paged_lane_row(int j, int u, int rg, int rpw, int nc)
{
    int row = j + u * rpw + rg;
    return row < nc ? row : nc - 1;
}

// A workgroup of NWV waves: query q, rows 0 .. nk - 1 of keys and values (row_stride elements apart; PACKED: read more than once,
// else nontemporal loads), position qpos.  knew / vnew (nullable): row nk - 1, which is stored into the cache here; they and q may
// be in LDS.  store(c, o) is called once per feature c.  PAGED: kp and vp are not read, rows come from the blocks that `tbl` lists
// (kvbuf: the pool).  s_bias: LDS for the head's table.  `early`: NoEarly, or (EarlyRows) the rows of
// the first step, for a caller that has also filled the table where it fits.  Uses barriers: every thread of the workgroup calls it.
struct NoEarly { static constexpr bool value = false; };
template <int U> struct EarlyRows { static constexpr bool value = true; uint4 k[U], v[U]; };
template <typename T, int DH, bool PACKED, int NWV, int U, bool PAGED, typename Store, typename Early = NoEarly>
__device__ __forceinline__ void attn_row_body(const T* qp, const T* kp, const T* vp, const T* knew, const T* vnew, int64_t row_stride,
                                              int nk, int qpos, int h, int H, float scale, const float* __restrict__ bias_by_dist,
                                              int radius, const T* kvbuf, const int32_t* __restrict__ tbl, int block_shift, float (&s_bias)[ATTN_BIAS_LDS],
                                              Store store, const Early& early = Early{})
{
    constexpr int EPL = 16 / sizeof(T);      // elements per 16-byte chunk
    constexpr int LPR = DH / EPL;            // lanes that share one key/value row
    constexpr int RPW = 64 / LPR;            // rows per wave per load
    constexpr int NL = (PAGED && RPW * U > 8) ? U : 1;   // PAGED: table look-ups per step
    static_assert(RPW <= 8, "the rows of one load must fit the smallest block");
    __shared__ float s_m[NWV], s_l[NWV];
    __shared__ __align__(16) float s_acc[NWV][DH];
    int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int rg = lane / LPR, cl = lane % LPR;
    // PAGED: keys of block b for this head start at block_k(b), its values H * block_rows * DH elements further on
    const int block_rows = 1 << block_shift;
    auto block_k = [&](int b) { return kvbuf + ((int64_t)b * 2 * H + h) * block_rows * DH; };
    // Fused append: the newest position's key/value rows come from the projection output; one 16-lane group
    // stores them into the cache, and every lane that meets row nk-1 reads it from the source instead of the
    // cache, so no ordering between that store and the loads is needed.
    if (!PACKED && knew) {
        if (wave == 0 && rg == 0) {
            const T *kd = kp, *vd = vp;
            int row = nk - 1;
            if (PAGED) {
                kd = block_k(tbl[row >> block_shift]);
                vd = kd + (int64_t)H * block_rows * DH;
                row &= block_rows - 1;
            }
            *(uint4*)(const_cast<T*>(kd) + (int64_t)row * DH + cl * EPL) = *(const uint4*)(knew + cl * EPL);
            *(uint4*)(const_cast<T*>(vd) + (int64_t)row * DH + cl * EPL) = *(const uint4*)(vnew + cl * EPL);
        }
    }

    float qf[EPL];
    {
        float t[EPL];
        Chunk<T, EPL>::unpack(*(const uint4*)(qp + cl * EPL), t);
#pragma unroll
        for (int e = 0; e < EPL; ++e) qf[e] = t[e] * scale * LOG2E;
    }
    const float* bias = bias_by_dist ? bias_by_dist + (int64_t)h * (2 * radius + 1) + radius : nullptr;
    // The head's bias table goes to LDS first (scaled for exp2): a look-up in global memory shares the wave's
    // in-order load counter with the K/V stream and cost 12 % of the kernel's bandwidth.
    const bool bias_lds = bias && 2 * radius + 1 <= ATTN_BIAS_LDS;
    if (bias_lds && !Early::value) {
        for (int i = threadIdx.x; i < 2 * radius + 1; i += NWV * 64) s_bias[i] = bias[i - radius] * LOG2E;
        __syncthreads();
    }
    auto bias_at = [&](int rel) {
        rel = rel < -radius ? -radius : (rel > radius ? radius : rel);
        return bias_lds ? s_bias[rel + radius] : bias[rel] * LOG2E;
    };

    float m_run = -INFINITY, l_run = 0.f, acc[EPL];
#pragma unroll
    for (int e = 0; e < EPL; ++e) acc[e] = 0.f;

    // with a fused append the cached rows are 0 .. nk-2; the new row is folded in after the loop
    const int nc = (!PACKED && knew) ? nk - 1 : nk;
    // PAGED: the blocks of a step are looked up one step ahead, so that the step's loads do not wait for the table.
    // Look-up x of the step starting at row j serves the rows of loads x, x + NL, ...; it names the block of row
    // min(j + x * RPW, nc - 1), which is also the block of every row those loads touch: rows past the end are
    // clamped to row nc - 1.
    int blk[NL];
    auto lookup = [&](int j) {
#pragma unroll
        for (int x = 0; x < NL; ++x) blk[x] = tbl[paged_lookup_row(j, x, RPW, nc) >> block_shift];
    };
    if (PAGED && wave * RPW * U < nc) lookup(wave * RPW * U);
    const int64_t v_off = PAGED ? (int64_t)H * block_rows * DH : vp - kp;        // values behind the keys
    for (int j0 = wave * RPW * U; j0 < nc; j0 += NWV * RPW * U) {
        uint4 kc[U], vc[U];
        float s[U];
        const T* kpb[NL];                     // PAGED: keys of this head in the block of look-up x
        int jb[NL];                           // PAGED: first row of that block
        kpb[0] = kp;
        jb[0] = 0;
        if (PAGED) {
#pragma unroll
            for (int x = 0; x < NL; ++x) {
                kpb[x] = block_k(blk[x]);
                jb[x] = paged_lookup_row(j0, x, RPW, nc) & ~(block_rows - 1);
            }
            int jn = j0 + NWV * RPW * U;
            if (jn < nc) lookup(jn);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            int x = NL == 1 ? 0 : u;
            int jj = paged_lane_row(j0, u, rg, RPW, nc) - jb[x];
            const T* kr = kpb[x] + (int64_t)jj * row_stride + cl * EPL;
            if constexpr (Early::value) {
                if (j0 < NWV * RPW * U) {
                    kc[u] = early.k[u];
                    vc[u] = early.v[u];
                    continue;
                }
            }
            kc[u] = load_chunk<!PACKED>(kr);
            vc[u] = load_chunk<!PACKED>(kr + v_off);
        }
        float mx = m_run;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float kf[EPL];
            Chunk<T, EPL>::unpack(kc[u], kf);
            float d = 0.f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) d = fmaf(qf[e], kf[e], d);
            d = row_sum<LPR>(d);
            int j = j0 + u * RPW + rg;
            if (bias) d += bias_at(j - qpos);
            s[u] = j < nc ? d : -INFINITY;
            mx = fmaxf(mx, s[u]);
        }
        float mref = mx == -INFINITY ? 0.f : mx;
        float alpha = fast_exp2(m_run - mref);
        l_run *= alpha;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] *= alpha;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            float p = fast_exp2(s[u] - mref);
            l_run += p;
            float vf[EPL];
            Chunk<T, EPL>::unpack(vc[u], vf);
#pragma unroll
            for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e]);
        }
        m_run = mx;
    }

    // the appended position (its key and value come from the projection output): folded into the state of the
    // first row group of wave 0
    if (!PACKED && knew && wave == 0 && rg == 0) {
        float kf[EPL], vf[EPL];
        Chunk<T, EPL>::unpack(*(const uint4*)(knew + cl * EPL), kf);
        Chunk<T, EPL>::unpack(*(const uint4*)(vnew + cl * EPL), vf);
        float d = 0.f;
#pragma unroll
        for (int e = 0; e < EPL; ++e) d = fmaf(qf[e], kf[e], d);
        d = row_sum<LPR>(d);
        if (bias) d += bias_at(nk - 1 - qpos);
        float mx = fmaxf(m_run, d);
        float alpha = fast_exp2(m_run - mx), p = fast_exp2(d - mx);
        l_run = l_run * alpha + p;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = fmaf(p, vf[e], acc[e] * alpha);
        m_run = mx;
    }

    // Merge the partial states: the row groups of a wave across its lanes, then the waves through LDS.  (All NWV * RPW states
    // through LDS, added up by DH threads, took 2-4 us of every launch.)
    auto merge_lanes = [&](auto xo) {
        constexpr int O = decltype(xo)::value;
        float mo = lane_xor<O>(m_run), lo = lane_xor<O>(l_run);
        float mx = fmaxf(m_run, mo), mref = mx == -INFINITY ? 0.f : mx;
        float wa = fast_exp2(m_run - mref), wb = fast_exp2(mo - mref);       // 0 for a side that saw no key
        l_run = l_run * wa + lo * wb;
#pragma unroll
        for (int e = 0; e < EPL; ++e) acc[e] = acc[e] * wa + lane_xor<O>(acc[e]) * wb;
        m_run = mx;
    };
    if constexpr (LPR <= 8) merge_lanes(std::integral_constant<int, 8>{});
    if constexpr (LPR <= 16) merge_lanes(std::integral_constant<int, 16>{});
    if constexpr (LPR <= 32) merge_lanes(std::integral_constant<int, 32>{});
    if (lane == 0) { s_m[wave] = m_run; s_l[wave] = l_run; }
    if (rg == 0) {
#pragma unroll
        for (int e = 0; e < EPL; e += 4) *(f32x4*)&s_acc[wave][cl * EPL + e] = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
    }
    __syncthreads();
    for (int c = threadIdx.x; c < DH; c += NWV * 64) {
        float M = s_m[0];
#pragma unroll
        for (int g = 1; g < NWV; ++g) M = fmaxf(M, s_m[g]);
        float L = 0.f, o = 0.f;
#pragma unroll
        for (int g = 0; g < NWV; ++g) {
            float w = fast_exp2(s_m[g] - M);      // 0 for waves that saw no key
            L += s_l[g] * w;
            o += s_acc[g][c] * w;
        }
        store(c, from_f32<T>(o / L));
    }
}

}  // namespace exe
