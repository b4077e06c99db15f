// Internal declarations shared by the HIP translation units of liblaps (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/laps.h"

typedef unsigned short bf16_t;  // storage: upper half of a float32
typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;

static __device__ __forceinline__ float bf16_to_f32(bf16_t b) { return __uint_as_float(((unsigned)b) << 16); }
static __device__ __forceinline__ bf16_t f32_to_bf16(float f) {
    __bf16 h = (__bf16)f;  // v_cvt_pk_bf16_f32: round-to-nearest-even
    return __builtin_bit_cast(bf16_t, h);
}
static __device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi) {
    return (unsigned)f32_to_bf16(lo) | ((unsigned)f32_to_bf16(hi) << 16);
}

void laps_set_error(const char* fmt, ...);
#define LAPS_HIP(call)                                                                         \
    do {                                                                                       \
        hipError_t e_ = (call);                                                                \
        if (e_ != hipSuccess) {                                                                \
            laps_set_error("%s failed: %s (%s:%d)", #call, hipGetErrorString(e_), __FILE__, __LINE__); \
            return LAPS_EHIP;                                                                  \
        }                                                                                      \
    } while (0)
#define LAPS_TRY(x)                 \
    do {                            \
        int rc_ = (x);              \
        if (rc_ != LAPS_OK) return rc_; \
    } while (0)
#define LAPS_LAUNCH_CHECK()                                                                    \
    do {                                                                                       \
        hipError_t e_ = hipGetLastError();                                                     \
        if (e_ != hipSuccess) {                                                                \
            laps_set_error("kernel launch failed: %s (%s:%d)", hipGetErrorString(e_), __FILE__, __LINE__); \
            return LAPS_EHIP;                                                                  \
        }                                                                                      \
    } while (0)

// ----------------------------------------------------------------------------- GEMM
// C = A[M,K] * W[N,K]^T, bf16 operands, fp32 accumulation, K-split into `split` slices.
enum GemmEpi {
    EPI_PARTIAL = 0,  // out_f32[split][M][N] raw partial sums
    EPI_RESID = 1,    // out_f32[M][N] = resid[M][N] + C              (single K slice only)
    EPI_SWIGLU = 2,   // out_bf16[M][N/2] = silu(gate) * up on interleaved columns (single K slice only)
};
struct GemmPlan {
    int cfg;          // tile shape index (see kTiles in gemm.hip)
    int split;        // K slices
    int k_per_split;  // multiple of 64
    int epi;          // epilogue the launch will apply: the requested one if split == 1, else EPI_PARTIAL
    int ws;           // slabs that every K slice holds a multiple of: 1 or 2
    int rest;         // 0, or 1 + the tile shape of the columns that whole rounds of `cfg` over the compute units leave
};
// partial_cap: bytes the partial sums of an automatic split may take above 128 rows or at K >= 2^22 (the layer driver
// passes what its workspace holds if that is less).
// row_kernel: a row kernel follows whether K is split or not and would add the slices as well: in a layer the RMSNorm
// behind a residual projection, or the kernel that takes raw sums.  False for a product of its own.
// layer: a projection inside a layer, which may take every tile.
constexpr size_t LAPS_PARTIAL_CAP = (size_t)256 << 20;
GemmPlan laps_gemm_plan(int m, int n, int k, int force_split, int want_epi, size_t partial_cap = LAPS_PARTIAL_CAP,
                        bool row_kernel = false, bool layer = false);
size_t laps_gemm_partial_bytes(int m, int n, int k, size_t partial_cap);
void laps_gemm_tile_dims(int cfg, int* bm, int* bn);   // rows and columns of tile shape `cfg` (0, 0 if unknown)
// row_live: NULL, or m entries; a negative entry marks a padding row.  Output rows of padding are unspecified; a row tile of
// padding only is skipped, and the tiles whose slabs go straight into LDS load no padding row at all.
// n_live: NULL, or a device int: rows at and past it are padding (batches whose padding is all at the end).
// live_varies: the launch will be replayed with other values of *n_live (a captured graph).
int laps_gemm_launch(const GemmPlan& p, const bf16_t* a, const bf16_t* w, int m, int n, int k, float* out_f32,
                     const float* resid, bf16_t* out_bf16, const int* row_live, const int* n_live, bool live_varies,
                     hipStream_t s);

// ----------------------------------------------------------------------------- element-wise / epilogues
int laps_launch_rope_table(float2* table, int max_pos, int head_dim, float theta, hipStream_t s);
// n_pool_pages (here, in the K/V movers and in the attention): page ids outside [0, n_pool_pages) are treated as
// unset entries - no cache write, no wild read.  INT_MAX when the caller has not said how many pages its pools hold.
// Begin of an un-captured batch: clamped lengths, attention work-item table (and shares); for each of n_rows rows (0: the
// attention alone, rows and first layer unused) its position and cache slot (page * 16 + offset, -1: padding or no
// cache write) and its RMSNorm with the first layer's gain.
struct BeginArgs {
    const int *row_start, *seq_len, *prefix_len, *page_table;   // seq_len may be NULL
    int n_seq, n_rows, max_pages, n_pool_pages;
    int group, rows_per_wg, max_items, n_kv, attn_wgs;          // attention blocking; attn_wgs as laps_attn_persistent_wgs
    int n_split, min_tiles;                                     // as laps_attn_plan
    int *new_len, *tok_pos, *tok_slot, *tile_start, *item_seq, *attn_pre;
    int4 *attn_bounds, *attn_desc;
    const float* x;
    const bf16_t* ln_w;
    bf16_t* r0;
    int d;
    float eps;
};
int laps_launch_begin(const BeginArgs& a, hipStream_t s);
// row_live (here and below): NULL, or one entry per row; rows with a negative entry are padding and are skipped.
int laps_launch_rmsnorm(const float* x, const bf16_t* w, bf16_t* out, int rows, int d, float eps, const int* row_live,
                        hipStream_t s);
// x_out = resid + sum_s partial[s]; if ln_w: r_out = rmsnorm(x_out; ln_w) in bf16.
int laps_launch_epi_resid(const float* partial, int split, const float* resid, float* x_out, const bf16_t* ln_w,
                          bf16_t* r_out, int rows, int d, float eps, const int* row_live, hipStream_t s);
int laps_launch_epi_qkv(const float* partial, int split, const bf16_t* bias, const int* tok_pos, const int* tok_slot,
                        const float2* rope, int max_pos, bf16_t* q_out, bf16_t* k_pool, bf16_t* v_pool, int rows,
                        int n_q, int n_kv, int hd, hipStream_t s);
int laps_launch_epi_swiglu(const float* partial, int split, bf16_t* act, int rows, int inter, const int* row_live,
                           hipStream_t s);
int laps_launch_pack_gate_up(const bf16_t* wg, const bf16_t* wu, bf16_t* dst, int inter, int d, hipStream_t s);
int laps_launch_kv_move(bool scatter, int n_seq, int n_tokens, const int* cu, const int* start_pos,
                        const int* page_table, int max_pages, bf16_t* k_tok, bf16_t* v_tok, bf16_t* k_pool,
                        bf16_t* v_pool, int n_kv, int hd, int n_pool_pages, hipStream_t s);
// Graph staging, one launch that leaves a captured stack nothing to prepare.  One workgroup writes the clamped lengths /
// prefixes of `depth` slots (the first n_real from the caller's device arrays, the rest empty), packed row offsets
// row_start_out[depth + 1], and the attention's work-item table for them; one workgroup per graph row its token position
// and cache slot (as laps_launch_begin), the row's input copied from x_rows (rows below n_rows; NULL: the graph's input
// rows are used as they are) into x_in, its RMSNorm with the first layer's gain into r0, and a share of the page-table
// copy (entries past n_real rows become 0).
struct StageArgs {
    const int *seq_len, *prefix_len, *page_table;   // caller's device arrays: [n_real], [n_real], [n_real][max_pages]
    const float* x_rows;                            // caller's packed input rows or NULL
    int n_real, n_rows, depth, len_bucket, max_pages, n_pool_pages;
    int group, rows_per_wg, max_items;              // attention blocking of the graph's shape
    int n_kv, attn_wgs;                             // workgroups of the persistent attention kernel (0: not used)
    int n_split, min_tiles;                         // as laps_attn_plan
    int *seq_len_out, *prefix_out, *row_start_out, *page_table_out;   // the graph's staging block
    int *new_len_out, *tok_pos, *tok_slot, *tile_start, *item_seq;    // the graph's workspace
    int* attn_pre;
    int4 *attn_bounds, *attn_desc;
    float* x_in;
    const bf16_t* ln_w;
    bf16_t* r0;
    int d;
    float eps;
};
int laps_launch_stage(const StageArgs& a, hipStream_t s);

// Inclusive prefix sum over a workgroup of 256 threads, and its total; sums: 4 ints of LDS.  Every thread calls it.
static __device__ __forceinline__ int laps_dev_scan(int v, int* sums, int* total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int up = __shfl_up(v, o, 64);
        if (lane >= o) v += up;
    }
    __syncthreads();   // sums may still be read from a previous call
    if (lane == 63) sums[wave] = v;
    __syncthreads();
    int before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        if (w < wave) before += sums[w];
        all += sums[w];
    }
    *total = all;
    return before + v;
}

// Work-item table of the attention for one batch: per-sequence number of query-row blocks, their exclusive prefix
// sum (tile_start[n_seq + 1]) and the sequence of every work item.  Runs in ONE workgroup of 256 threads; sums: 4 ints
// of LDS.  Shared by the kernel that begins a batch and the staging kernel of graphs.
static __device__ __forceinline__ void laps_dev_attn_sched(const int* __restrict__ new_len, int n_seq, int group,
                                                           int rows_per_wg, int* __restrict__ tile_start,
                                                           int* __restrict__ item_seq, int max_items, int* sums) {
    int done = 0;   // items of the sequences before
    for (int base = 0; base < n_seq; base += 256) {
        const int i = base + threadIdx.x;
        const int v = (i < n_seq) ? (new_len[i] * group + rows_per_wg - 1) / rows_per_wg : 0;
        int total;
        const int first = done + laps_dev_scan(v, sums, &total) - v;
        if (i < n_seq) {
            tile_start[i] = first;
            // bound: lengths that disagree with the row offsets must not write past the table
            for (int k = 0; k < v && first + k < max_items; ++k) item_seq[first + k] = i;
        }
        done += total;
    }
    if (threadIdx.x == 0) tile_start[n_seq] = done;
}

// A prefix length that the page table cannot hold (a corrupted or stale array) must neither index past the
// table nor make a workgroup walk millions of key tiles: cut to what max_pages pages can address.
static __device__ __forceinline__ int laps_dev_clamp_prefix(int h, int new_len, int max_pages) {
    const int room = max_pages * LAPS_PAGE - new_len;
    h = h < room ? h : room;
    return h > 0 ? h : 0;
}

constexpr int LAPS_ATTN_KT = 64;          // keys per tile

// What a workgroup of the attention needs to know of a work item, two int4 an item: (sequence, row block, new tokens, cached
// tokens) and (first row, parts of its key range, key tiles of a part, -); the items past the batch's last one have a sequence of
// -1.  One scalar load instead of the chain item -> sequence -> lengths -> first row, at 0.3 to 0.5 us a link.
// Key-range splits of a batch whose (item, kv head) blocks leave compute units idle (n_split > 1): an item's key tiles go out in
// parts of equal length, at least min_tiles each and n_split of them at most.  Where an item is cut follows from its own length and
// the launch's shape alone, so that the bits of a request do not depend on the lengths it is batched with.  (Parts of equal length
// over the whole batch would spare the longest item's parts, 32B, turns of 17 to 32 tokens over 512 to 4096 keys, up to 9 tiles
// where all parts together are 4 tiles for every place on the chip: a layer's graph 252 -> 247 us.  They need a table of the parts:
// written by the items' threads, 15 parts of one turn took 5 us.)
// Runs in ONE workgroup of 256 threads after laps_dev_attn_sched.
static __device__ __forceinline__ void laps_dev_attn_desc(const int* __restrict__ new_len, const int* __restrict__ prefix_len,
                                                          const int* __restrict__ row_start, int n_seq, int group, int rows_per_wg,
                                                          int max_pages, const int* tile_start, const int* item_seq, int max_items,
                                                          int n_split, int min_tiles, int4* __restrict__ desc) {
    __syncthreads();   // tile_start and item_seq were written by other threads of this workgroup
    const int total = tile_start[n_seq];
    for (int k = threadIdx.x; k < max_items; k += 256) {
        const bool any = k < total;
        const int i = any ? item_seq[k] : 0, L = new_len[i], H = laps_dev_clamp_prefix(prefix_len[i], L, max_pages), q = any ? k - tile_start[i] : 0;
        int parts = 1, each = 0;
        if (n_split > 1 && any) {
            const int last = ((q + 1) * rows_per_wg < L * group ? (q + 1) * rows_per_wg : L * group) - 1;
            const int nt = (H + last / group + LAPS_ATTN_KT) / LAPS_ATTN_KT, most = nt / min_tiles < n_split ? nt / min_tiles : n_split;
            each = most > 1 ? (nt + most - 1) / most : nt;
            parts = (nt + each - 1) / each;   // none of them empty
        }
        desc[2 * k] = any ? make_int4(i, q, L, H) : make_int4(-1, 0, 0, 0);
        desc[2 * k + 1] = make_int4(row_start[i], parts, each, 0);
    }
}

// Equal shares of a batch's attention for `n_wgs` workgroups (the persistent long-prompt kernel).  A unit is one
// (kv head, work item) pair and costs its key tiles plus COST0 (its prologue and epilogue; 1 to 10 tried, 4 is best or even); the units
// of all kv heads, one head after the other, are cut into equal lengths.  bounds[w] = (kv head, item, first tile) is
// where workgroup w begins and w - 1 ends.  A cut inside a unit stays MIN_SEG tiles clear of its ends and where every
// row of the unit sees the first key after the cut, else it moves to the unit's begin or end; short batches use fewer
// workgroups, spread over the compute units.  Where every unit has a workgroup to itself and the longest is no longer
// than a share with what cutting costs (partial results, their merge, uneven cuts), nothing is cut: 32B shape, 16 short
// turns (176 units of 5) 32 us in shares of several units, 23 so; 16 turns over up to 1472 keys (units of up to 27, shares
// of 11) 55 us cut, 63 not; 1000 rows over 600 (160 units of up to 30, shares of 13) 73 cut, 66 not.
// Runs in ONE workgroup of 256 threads after laps_dev_attn_sched; pre (max_items + 1 ints) holds the prefix sums of the
// item costs.
constexpr int LAPS_ATTN_LONG_ROWS = 256;  // query rows per work item of the long-prompt kernel
constexpr int LAPS_ATTN_MAX_WGS = 256;    // one workgroup per compute unit
constexpr int LAPS_ATTN_COST0 = 4;        // in key tiles (about 2 us), as CUT_COST
static __device__ __forceinline__ void laps_dev_attn_bounds(const int* __restrict__ new_len,
                                                            const int* __restrict__ prefix_len, int n_seq, int group,
                                                            int n_kv, int max_pages, const int* tile_start,
                                                            const int* item_seq, int max_items, int n_wgs, int* pre,
                                                            int4* bounds, int* sums) {
    constexpr int COST0 = LAPS_ATTN_COST0, MIN_SEG = 4, MIN_COST = 8, CUT_COST = 14;
    __syncthreads();   // tile_start and item_seq were written by other threads of this workgroup
    const int total = tile_start[n_seq], n_items = total < max_items ? total : max_items;
    // key tiles of an item, and the last tile a cut may begin with
    auto tiles_of = [&](int i, int* last_cut) {
        const int seq = item_seq[i], L = new_len[seq], H = laps_dev_clamp_prefix(prefix_len[seq], L, max_pages);
        const int r0 = (i - tile_start[seq]) * LAPS_ATTN_LONG_ROWS, rows = L * group;
        const int last = (r0 + LAPS_ATTN_LONG_ROWS < rows ? r0 + LAPS_ATTN_LONG_ROWS : rows) - 1;
        *last_cut = (H + r0 / group) / LAPS_ATTN_KT;
        return (H + last / group + LAPS_ATTN_KT) / LAPS_ATTN_KT;
    };
    if (threadIdx.x == 0) pre[0] = 0;
    int per_head = 0, longest = 0;   // cost of the items, and of the longest one this thread, then any, sees
    for (int base = 0; base < n_items; base += 256) {
        const int i = base + threadIdx.x;
        int unused, total_cost;
        const int own = i < n_items ? tiles_of(i, &unused) + COST0 : 0;
        longest = own > longest ? own : longest;
        const int upto = per_head + laps_dev_scan(own, sums, &total_cost);
        if (i < n_items) pre[i + 1] = upto;
        per_head += total_cost;
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const int other = __shfl_xor(longest, o, 64);
        longest = other > longest ? other : longest;
    }
    __syncthreads();   // sums are read
    if ((threadIdx.x & 63) == 0) sums[threadIdx.x >> 6] = longest;
    __syncthreads();   // and pre is written
    for (int w = 0; w < 4; ++w) longest = sums[w] > longest ? sums[w] : longest;
    const long cost = (long)per_head * n_kv, units = (long)n_items * n_kv;
    const bool cut = units > n_wgs || longest > cost / n_wgs + CUT_COST;
    long share = cost / MIN_COST;   // as many workgroups get one, but no fewer than there are units
    share = !cut || share < units ? units : share;
    share = share < 1 ? 1 : (share > n_wgs ? n_wgs : share);
    const int used = (int)share;
    for (int w = threadIdx.x; w <= n_wgs; w += 256) {
        int4 b = make_int4(n_kv, 0, 0, 0);   // the end
        const int u = (w * used + n_wgs - 1) / n_wgs;   // share w begins where the u-th of `used` equal ones does
        // 64-bit quotients take a microsecond
        const long x = u >= used ? cost : cost < (1 << 22) ? (long)((unsigned)cost * (unsigned)u / (unsigned)used) : cost * u / used;
        if (!cut) {
            if (u < units) b = make_int4(u / n_items, u % n_items, 0, 0);
        } else if (x < cost) {
            const int head = cost < (1 << 22) ? (int)((unsigned)x / (unsigned)per_head) : (int)(x / per_head), rem = (int)(x - (long)head * per_head);
            int lo = 0, hi = n_items;   // item with pre[item] <= rem < pre[item + 1]
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (pre[mid] <= rem) lo = mid; else hi = mid;
            }
            int last_cut;
            const int nt = tiles_of(lo, &last_cut);
            int t = rem - pre[lo] - COST0;
            if (t < MIN_SEG) t = 0;
            const bool next = t > 0 && (t > last_cut || nt - t < MIN_SEG);
            if (!next) b = make_int4(head, lo, t, 0);
            else if (lo + 1 < n_items) b = make_int4(head, lo + 1, 0, 0);
            else b = make_int4(head + 1, 0, 0, 0);   // head + 1 == n_kv: the end
        }
        bounds[w] = b;
    }
}

// ----------------------------------------------------------------------------- attention
// The work-item table is made with the blocking of the same (n_seq, n_tokens, max_pages) (laps_attn_plan).
// `partial` (partial_bytes >= laps_attn_partial_bytes, 16-byte aligned) receives per-split results when the launch shape
// calls for splitting the key range; it may be NULL only if max_pages * 16 < 512.  partial_bytes must be that of the table's shares.
// tile_start: n_seq + 1 ints; item_seq: laps_attn_item_table_bytes (sequence of every row-block work item).
size_t laps_attn_partial_bytes(int hd, int max_pages);   // 0 when page tables this narrow never split
// Work-item table: item_seq, then the cost prefix sums and the bounds of the persistent kernel and the items' descriptions.
size_t laps_attn_item_table_bytes(int max_tokens, int max_seqs, int group);
void laps_attn_item_tables(int* item_seq, int n_tokens, int n_seq, int group, int** pre, int4** bounds, int4** desc);
// Workgroups of the persistent long-prompt kernel for a launch shape with partial_bytes of room for the results of cut
// units (two slots per workgroup); 0: the launch does not use it.
int laps_attn_persistent_wgs(int n_seq, int n_tokens, int group, int n_kv, int hd, int max_pages, size_t partial_bytes);
// The blocking laps_launch_attention derives from a launch shape, for the work-item table: query rows per workgroup,
// bound on the (sequence, row block) items, key-range splits (1 = none), fewest key tiles a split may get.
void laps_attn_plan(int n_seq, int n_tokens, int group, int n_kv, int max_pages, int* rows_per_wg, int* max_items,
                    int* n_split, int* min_tiles_per_split);
// Lengths and row offsets are those that the kernel which began or staged the batch has put into the table.
int laps_launch_attention(const bf16_t* q, bf16_t* out, const bf16_t* k_pool, const bf16_t* v_pool,
                          const int* page_table, int max_pages, int n_seq, int n_tokens, const int* tile_start,
                          const int* item_seq, float* partial, size_t partial_bytes, int n_q, int n_kv, int hd, int n_pool_pages,
                          hipStream_t s);
