// Launchers of the gfx950 kernels.  All pointers are device pointers unless a comment says host.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <vector>

namespace exe {

// Where a projection's key / value features go instead of `out`: straight into the cache.  Feature n >= first_col of row m is
// element kv_at(row[m], cap[m], head0 + (n - first_col) / dh, dh_shift) + (n - first_col) % dh of `pool` (the keys of all heads, then
// the values), dh = 2^dh_shift; first_col is a multiple of 64.
struct KvStore {
    void* pool = nullptr;
    const int64_t* row = nullptr;
    const int32_t* cap = nullptr;
    int first_col = 0, dh_shift = 0, head0 = 0;
};
// row: the first element of the position in the extent's first head; cap * dh, the elements of a head, need not fit 32 bits
__host__ __device__ __forceinline__ int64_t kv_row_of(int64_t base, int pos, int dh) { return base + (int64_t)pos * dh; }
__host__ __device__ __forceinline__ int64_t kv_at(int64_t row, int cap, int head, int dh_shift) { return row + ((int64_t)head * cap << dh_shift); }

struct GemmArgs {
    int dtype;            // DT_F32 / DT_BF16: type of A, W, bias and (for OUT_T) out
    int M, N, K;
    const void* A;        // [M, K] row-major
    const void* W;        // [N, K] row-major
    const void* bias;     // [N] or nullptr
    int act;              // -1 none, 0 relu, 1 gelu(erf); applied in OUT_T mode
    float alpha;          // result = alpha * (A.W^T) + bias
    int out_mode;         // OUT_T, OUT_RESID (float out += result), OUT_F32
    void* out;            // [M, N]
    float* workspace;     // split-K partial sums
    size_t workspace_bytes;
    int lda = 0, ldw = 0; // row strides of A and W in elements (0 = K); the generic kernel takes dense rows only
    // Launches of few rows may run on the streaming kernel (the model's do; exe_op_gemm serves bf16 with the tile kernel
    // alone, whose launch plans exe_op_gemm_plan reports).
    bool few_rows = false;
    // OUT_RESID only: the caller's next kernel can add split-K partials to the residual stream itself.  launch_gemm then
    // leaves them in the workspace, *pending = their number (0: the result is complete), and plans with the cheaper split.
    int* pending = nullptr;
    // nullable, out_mode OUT_T without activation: stored so by the launches that can (gemm_kv_rows leading rows); the others'
    // features all go to `out`
    const KvStore* kv = nullptr;
    int force_cfg = -1, force_splits = 0;     // tile configuration and split-K parts in place of the planner's (gemm_force_ok)
};
// whether the tile kernels take bf16 shapes in a configuration (-1: any) and with a number of parts
bool gemm_force_ok(int cfg, int splits, int M, int N, int K);
enum GemmMode { GEMM_TILE_ONLY = 0, GEMM_FEW_ROWS = 1, GEMM_DEFER = 2 };       // flags, as the two members above
constexpr int MAX_SPLIT_ROWS = 4096;      // no launch of more rows is split over K
size_t gemm_workspace_bytes(int dtype, int M, int N, int K, int mode);
// how a shape is launched with few_rows = (dtype is float): route (0 tile kernel, 1 streaming kernel, 2 generic), tile configuration (0 64x256, 1 128x256, 2 256x256, 3 64x128,
// 4 128x128, 5 256x128, 6 192x256, 8 256x160), split-K parts, and the leading rows that the first launch takes (M unless the rows beyond
// whole rounds of tiles go to a second launch)
void gemm_plan_info(int dtype, int M, int N, int K, int* route, int* cfg, int* splits, int* rows_first);
hipError_t launch_gemm(const GemmArgs& a, hipStream_t s);
// the leading rows whose key / value features launch_gemm(a) stores through a.kv
int gemm_kv_rows(const GemmArgs& a);
// the launches of launch_gemm(a) in the order of their rows: how many there are, and of the first `cap` the rows and whether such a
// launch can store through a.kv
int gemm_launches(const GemmArgs& a, int cap, int32_t* rows, int32_t* stores);
// and five numbers of each as exe_op_gemm_model_plan has them
int gemm_launch_plans(const GemmArgs& a, bool defer, int cap, int32_t* plans);

// The streaming kernel (kernels_gemm_stream.hip): nt * 16 output features of ma * 8 rows per workgroup, K in `splits` parts of
// units_per_split units (128 bytes of a row each); nt = 0: a shape it does not take.  launch_gemm_stream leaves float
// partials in a.workspace if splits > 1.
struct StreamPlan { int nt = 0, ma = 0, splits = 1, units_per_split = 0; double cost = 0.0; };
StreamPlan gemm_stream_plan(int dtype, int M, int N, int K, bool defer);
StreamPlan gemm_stream_candidate(int dtype, int nt, int ma, int splits, int M, int N, int K, bool defer);    // nt in {1, 2, 4, 5}, ma in {1, 2, 4, 6, 8}
// The large tile kernel (kernels_gemm_large.hip, bf16): 256, 192 or 128 x 256, 256 x 160 or 256 x 128 tiles, persistent on at most grid_max
// workgroups, K in `splits` parts of k_per_split (every part at least 2 k-tiles of 64).
hipError_t launch_gemm_large(const GemmArgs& a, int bm, int bn, int k_per_split, int splits, int grid_max, hipStream_t s);
// The float tiles (kernels_gemm_f32.hip): K a multiple of 32, operands and bias 16-byte aligned.
hipError_t launch_gemm_f32(const GemmArgs& a, hipStream_t s);
int gemm_f32_tile(int M, int N, int K, double* seconds);       // 0 128 x 128, 1 64 x 128, 2 64 x 64
double gemm_f32_cost(int M, int N, int K);       // seconds
double stream_f32_seconds(const StreamPlan& p, int M, int N, int K);
hipError_t launch_splitk_reduce(const GemmArgs& a, int splits, hipStream_t s);
hipError_t launch_gemm_stream(const GemmArgs& a, const StreamPlan& p, hipStream_t s);

// A launch counts its threads in 32 bits, and takes more modulo 2^32 without an error.
constexpr int64_t MAX_LAUNCH_THREADS = 0xffffffff;

// A kernel's dynamic LDS limit, raised once per kernel and device.
constexpr int MAX_DEVICES = 64;
struct LdsLimit {
    std::once_flag once;
    hipError_t err = hipSuccess;
    hipError_t raise(const void* kern, int bytes)
    {
        std::call_once(once, [&]() { err = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
        return err;
    }
};

// copies a call's descriptors (16-byte aligned buffers of a multiple of 16 bytes) from pinned host memory
hipError_t launch_stage(const void* host, void* dev, size_t bytes, hipStream_t s);
hipError_t launch_embed(int dtype, const int32_t* tokens, const int32_t* pos, int T, int d, const void* tok_emb,
                        const void* pos_emb, float* h, hipStream_t s);
hipError_t launch_load_hidden(int dtype, const void* x, int64_t n, float* h, hipStream_t s);
hipError_t launch_store_hidden(int dtype, const float* h, int64_t n, void* out, hipStream_t s);
// The largest of 16 neighbouring features of a row and its index, [feature / 16][16 rows]; index 0x7fffffff: all NaN.
struct TopLogit { float value; int32_t index; };
struct NormArgs {
    int dtype, rms;
    float* x;                    // residual rows; written only with `partial`
    const int32_t* row_index;    // nullable: selects rows of x (and of the partials)
    int rows, d;
    const void *gain, *shift;    // shift: LayerNorm only
    float eps, out_scale;
    void* out;                   // [rows, d] in dtype
    // split-K partials [splits][partial_rows][d] of the projection that ends in x, and its bias (nullable): added to x first
    const float* partial = nullptr;
    int splits = 0, partial_rows = 0;
    const void* bias = nullptr;
    bool last = false;           // nothing reads x after this norm
    TopLogit* top = nullptr;     // launch_norm_gemm only (float outputs, no bias, alpha 1), may be pinned: see TopLogit
};
hipError_t launch_norm(const NormArgs& a, hipStream_t s);
// A norm and the product behind it in one launch of the streaming kernel (a.A is not read), where norm_gemm_fits says so.
bool norm_gemm_fits(const NormArgs& n, const GemmArgs& a);
hipError_t launch_norm_gemm(const NormArgs& n, const GemmArgs& a, hipStream_t s);
// ---- decode iterations of small models (kernels_small.hip): a layer's attention block and feed-forward block, a launch each
constexpr int SMALL_MAX_ROWS = 32, SMALL_MAX_PARTS = 64, SMALL_SLICE = 32;     // rows; heads, or slices of the feed-forward; features of a slice
bool small_decode_fits(int dtype, int rows, int d, int H, int dh, int f);
struct SmallArgs {               // the residual stream in front of a block, its norm, and where the block's partial sums go
    int dtype, rows, d, rms;
    float eps;
    const void *gain, *shift;    // shift: LayerNorm only
    const float* x;              // [rows, d]
    float* x_out;                // [rows, d], not x: the rows with the partial sums in front of the block added
    const float* partial;        // [n_part][rows][d], of the block in front, and its bias (nullable)
    int n_part;
    const void* part_bias;
    float* out;                  // [heads, or f / SMALL_SLICE][rows][d], not `partial`
    // attention only, nullable: the rows are these embeddings, x is not read
    const int32_t *tokens = nullptr, *pos = nullptr;
    const void *tok_emb = nullptr, *pos_emb = nullptr;
    // attention only, nullable: stage_bytes (as launch_stage takes them) that this launch copies for the launches behind it
    const void* stage_from = nullptr;
    void* stage_to = nullptr;
    size_t stage_bytes = 0;
};
struct SmallAttn {               // arrays as in AttnCacheArgs; self-attention appends the rows' keys and values at len - 1
    int H, dh, cross;
    const void *w_in, *b_in;     // [3 * H * dh, d], or (cross) [H * dh, d]; b_in nullable
    const void* w_out;           // [d, H * dh]
    void* pool;
    const int64_t* base; const int32_t* cap; const int32_t* len; const int32_t* qpos;
    int layer;
    float scale;
    const float* bias_by_dist; int bias_radius;
};
struct SmallFfn { int f; const void *w_1, *b_1; int act; const void* w_2; };     // b_1 nullable
hipError_t launch_small_attn(const SmallArgs& a, const SmallAttn& k, hipStream_t s);
hipError_t launch_small_ffn(const SmallArgs& a, const SmallFfn& k, hipStream_t s);
// copies K and V rows of `src` (row stride ld, K at column k_off, V at v_off) into the cache:
// token t belongs to batch entry tok_b[t] (t itself if nullptr) at position tok_pos[t];
// K of (b, head, pos) lives at pool + base[b] + ((layer*2+0)*H + head)*cap[b]*dh + pos*dh, V at kv index 1.
hipError_t launch_kv_append(int dtype, const void* src, int ld, int k_off, int v_off, int T, const int32_t* tok_b,
                            const int32_t* tok_pos, const int64_t* base, const int32_t* cap, int layer, int H, int dh,
                            void* pool, hipStream_t s);
hipError_t launch_kv_append_paged(int dtype, const void* src, int ld, int k_off, int v_off, int T, const int32_t* tok_b,
                                  const int32_t* tok_pos, const int32_t* table, int table_w, int shift, int H, int dh,
                                  void* layer_pool, hipStream_t s);
// row[t] and row_cap[t] of KvStore for token t of an encode batch, whose sequence tok_b[t] has the extent base, cap
hipError_t launch_kv_rows(const int32_t* tok_b, const int32_t* tok_pos, const int64_t* base, const int32_t* cap, int T, int dh,
                          int64_t* row, int32_t* row_cap, hipStream_t s);
hipError_t launch_argmax(const float* logits, int rows, int n, int32_t* out, hipStream_t s);

struct AttnCacheArgs {       // one query row per batch entry against that sequence's cached K/V
    int dtype, B, H, dh;
    const void* q; int q_stride;          // q of (b, head) at q + b*q_stride + head*dh
    const void* pool;
    const int64_t* base; const int32_t* cap; const int32_t* len; const int32_t* qpos;
    int layer;                             // K at base + ((layer*2)*H + head)*cap*dh
    float scale;
    const float* bias_by_dist; int bias_radius;   // [H, 2r+1] or nullptr
    void* out;                             // [B, H*dh]
    // fused append (optional): the new position's key / value rows of (b, head) are at
    // q + b*q_stride + new_k_off + head*dh and ... + new_v_off; the kernel stores them at position len-1 of the
    // cache and attends to them straight from there (new_k_off = 0 disables)
    int new_k_off = 0, new_v_off = 0;
    int mean_len = 0, max_len = 0;         // average and largest len of the batch (0 = unknown): pick the launch shape
};
hipError_t launch_attn_cache(const AttnCacheArgs& a, hipStream_t s);

struct AttnPagedArgs {       // as AttnCacheArgs, with the cache of one layer held in blocks of 2^block_shift positions
    int dtype, B, H, dh;
    const void* q; int q_stride;
    const void* pool;                      // block b at pool + b * 2*H*2^block_shift*dh elements: [K|V][head][row][dh]
    const int32_t* block_table; int max_blocks; int block_shift;    // [B, max_blocks]
    const int32_t* len; const int32_t* qpos;
    float scale;
    const float* bias_by_dist; int bias_radius;
    void* out;
    int new_k_off = 0, new_v_off = 0;      // fused append, as in AttnCacheArgs
    int mean_len = 0, max_len = 0;
};
hipError_t launch_attn_paged(const AttnPagedArgs& a, hipStream_t s);
// host-side replay of the paged kernel's row indexing (0 = every row read lies in its block and is read once)
int paged_index_check(int dtype, int dh, int block_shift, int nwv, int len);

constexpr int PREFILL_TILE_Q = 128, PREFILL_TILE_K = 64;
struct PrefillWork {         // of one head over a batch
    int max_len = 0;         // longest sequence
    int64_t pairs = 0;       // (query row, key) pairs
    int64_t key_tiles = 0;   // key tiles of all query tiles
};
PrefillWork prefill_work(const int32_t* lens, int n_seqs, bool causal);
struct AttnPackedArgs {      // ragged prefill over packed qkv [T, 3*H*dh]
    int dtype, T, H, dh, n_seqs;
    const void* qkv;
    const int32_t* tok_b;    // [T] sequence index of each token
    const int32_t* tok_pos;  // [T] position in its sequence
    const int32_t* cu;       // [n_seqs+1] first token of each sequence
    int causal;
    float scale;
    const float* bias_by_dist; int bias_radius;
    void* out;               // [T, H*dh]
    // tile list for the MFMA kernel: (seq, first query row) pairs in the order prefill_tile_order gives
    const int32_t* tiles; int n_tiles;
    int force_generic;       // 0: the faster kernel for the batch's work; > 0 the row kernel, < 0 the MFMA kernel wherever it takes the call
    PrefillWork work;
    // nullable: keys and values come from the cache, as in AttnCacheArgs, instead of from qkv
    const void* pool = nullptr;
    const int64_t* base = nullptr; const int32_t* cap = nullptr;
    int layer = 0;
};
// Appends the (seq, first query row) pairs of a batch's 128-row query tiles to `tiles`: sequences longest first, the
// tiles of one sequence together, last rows (causal: most keys) first.  The tiles of a sequence read the same keys
// and values, and the kernel's workgroup numbering puts neighbours of this list (for one head) on one XCD at about
// the same time, so that they arrive in that XCD's L2 once; longest first keeps the short work for the end of the
// launch.  (Measured against most-work-first over the whole batch and over groups of 8 to 40 tiles: this order is
// the fastest or within 1 % of it on ragged and uniform batches, and halves the kernel's HBM reads.)
void prefill_tile_order(const int32_t* lens, int n_seqs, std::vector<int32_t>& tiles);
hipError_t launch_attn_packed(const AttnPackedArgs& a, hipStream_t s);

}  // namespace exe
