// Row-wise kernels around the GEMMs: token metadata, RMSNorm, split-K reductions fused with the
// layer's element-wise steps (residual + next RMSNorm, RoPE + KV append, SwiGLU), weight packing
// and KV cache moves.  All are bandwidth-trivial next to the GEMMs; they use one workgroup per
// row with 16-byte accesses.
#include <type_traits>

#include "laps_internal.h"

namespace {

constexpr int ROW_THREADS = 256;

__device__ __forceinline__ float block_sum(float v, float* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    __syncthreads();  // red may still be read from a previous call
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < ROW_THREADS / 64; ++w) t += red[w];
    return t;
}

// ------------------------------------------------------------------ rope table (fp64 evaluation)
__global__ void rope_table_kernel(float2* table, int max_pos, int half, double theta, int hd) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= max_pos * half) return;
    const int p = i / half, j = i % half;
    const double inv_freq = pow(theta, -2.0 * (double)j / (double)hd);
    const double ang = (double)p * inv_freq;
    table[i] = make_float2((float)cos(ang), (float)sin(ang));
}

// ------------------------------------------------------------------ token metadata
// Owning sequence of a row by binary search over row_start, then absolute position and KV slot
// (page * 16 + offset) of the token; -1 for padding rows.
__device__ __forceinline__ void token_meta(int row, int n_seq, const int* __restrict__ row_start,
                                           const int* __restrict__ seq_len, const int* __restrict__ prefix_len,
                                           const int* __restrict__ page_table, int max_pages, int n_pool_pages, int* pos_out,
                                           int* slot_out) {
    int lo = 0, hi = n_seq;  // find s with row_start[s] <= row < row_start[s+1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (row_start[mid] <= row) lo = mid; else hi = mid;
    }
    const int s = lo;
    const int t = row - row_start[s];
    const int cap = row_start[s + 1] - row_start[s];
    int l = seq_len ? seq_len[s] : cap;
    l = l > cap ? cap : l;
    int pos = -1, slot = -1;
    if (t >= 0 && t < l) {
        const int h = prefix_len[s];
        pos = (h > 0 ? h : 0) + t;
        // a position past the table's width, an unset (-1) entry or a page id outside the pool: no cache write
        const int pi = pos / LAPS_PAGE;
        const int page = pi < max_pages ? page_table[(size_t)s * max_pages + pi] : -1;
        slot = (page >= 0 && page < n_pool_pages) ? page * LAPS_PAGE + pos % LAPS_PAGE : -1;
    }
    *pos_out = pos;
    *slot_out = slot;
}

// ------------------------------------------------------------------ RMSNorm: fp32 row -> bf16 row
// One row of d <= 4 * ROW_THREADS * MAXV values with ROW_THREADS threads, held in registers between the two passes; red
// holds ROW_THREADS / 64 floats of LDS.
constexpr int ROW_MAXV = 8192 / 4 / ROW_THREADS;
template <int MAXV>
struct RowRegs {
    f32x4 v[MAXV];
    u32x2 gain[MAXV];   // loaded with the row: behind the reduction they would be a second round trip
    __device__ __forceinline__ void load(const f32x4* __restrict__ xr, const bf16_t* __restrict__ w, int d) {
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            const int i = threadIdx.x + j * ROW_THREADS;
            if (i < d / 4) v[j] = xr[i], gain[j] = reinterpret_cast<const u32x2*>(w)[i];
        }
    }
    __device__ __forceinline__ void store(f32x4* __restrict__ dst, int d) const {
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            const int i = threadIdx.x + j * ROW_THREADS;
            if (i < d / 4) dst[i] = v[j];
        }
    }
    __device__ __forceinline__ void norm(bf16_t* __restrict__ out_row, int d, float eps, float* red) const {
        float ss = 0.f;
#pragma unroll
        for (int j = 0; j < MAXV; ++j)
            if (threadIdx.x + j * ROW_THREADS < d / 4) ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
        const float inv = rsqrtf(block_sum(ss, red) / (float)d + eps);
        u32x2* orow = reinterpret_cast<u32x2*>(out_row);
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            const int i = threadIdx.x + j * ROW_THREADS;
            if (i < d / 4) {
                const u32x2 g = gain[j];
                u32x2 o;
                o.x = pack_bf16x2(v[j].x * inv * __uint_as_float(g.x << 16), v[j].y * inv * __uint_as_float(g.x & 0xffff0000u));
                o.y = pack_bf16x2(v[j].z * inv * __uint_as_float(g.y << 16), v[j].w * inv * __uint_as_float(g.y & 0xffff0000u));
                orow[i] = o;
            }
        }
    }
};

template <int MAXV>
__global__ __launch_bounds__(ROW_THREADS) void rmsnorm_kernel(const float* __restrict__ x,
                                                               const bf16_t* __restrict__ w, bf16_t* __restrict__ out,
                                                               int d, float eps, const int* __restrict__ row_live) {
    __shared__ float red[ROW_THREADS / 64];
    const size_t row = blockIdx.x;
    if (row_live && row_live[row] < 0) return;  // padding row: nothing reads its output
    RowRegs<MAXV> r;
    r.load(reinterpret_cast<const f32x4*>(x + row * d), w, d);
    r.norm(out + row * d, d, eps, red);
}

// ------------------------------------------------------------------ begin of an un-captured batch
// Workgroup 0: clamped lengths and the attention's work-item table (and shares).  Workgroup 1 + r: row r's position and
// cache slot and its first RMSNorm.  All of it is latency: three launches one after the other took 4.7 + 8.1 + 7.4 us
// ahead of 573 rows of the 32B shape, this one 10.3 (2048 rows: 29 and 18).
template <int MAXV>
__global__ __launch_bounds__(ROW_THREADS) void begin_kernel(const BeginArgs a) {
    __shared__ int sums[ROW_THREADS / 64];
    __shared__ float red[ROW_THREADS / 64];
    __shared__ int row_pos;
    if (blockIdx.x == 0) {
        for (int i = threadIdx.x; i < a.n_seq; i += ROW_THREADS) {
            const int cap = a.row_start[i + 1] - a.row_start[i];
            int l = a.seq_len ? a.seq_len[i] : cap;
            l = l > cap ? cap : l;
            a.new_len[i] = l < 0 ? 0 : l;
        }
        __syncthreads();   // the lengths written above are read below by other threads of this workgroup
        laps_dev_attn_sched(a.new_len, a.n_seq, a.group, a.rows_per_wg, a.tile_start, a.item_seq, a.max_items, sums);
        laps_dev_attn_desc(a.new_len, a.prefix_len, a.row_start, a.n_seq, a.group, a.rows_per_wg, a.max_pages, a.tile_start, a.item_seq,
                           a.max_items, a.n_split, a.min_tiles, a.attn_desc);
        if (a.attn_wgs > 0)
            laps_dev_attn_bounds(a.new_len, a.prefix_len, a.n_seq, a.group, a.n_kv, a.max_pages, a.tile_start, a.item_seq,
                                 a.max_items, a.attn_wgs, a.attn_pre, a.attn_bounds, sums);
        return;
    }
    const int row = blockIdx.x - 1;
    RowRegs<MAXV> r;
    r.load(reinterpret_cast<const f32x4*>(a.x + (size_t)row * a.d), a.ln_w, a.d);
    if (threadIdx.x == 0) {
        int pos, slot;
        token_meta(row, a.n_seq, a.row_start, a.seq_len, a.prefix_len, a.page_table, a.max_pages, a.n_pool_pages, &pos, &slot);
        a.tok_pos[row] = pos;
        a.tok_slot[row] = slot;
        row_pos = pos;
    }
    __syncthreads();
    if (row_pos < 0) return;   // padding row: nothing reads its normed row
    r.norm(a.r0 + (size_t)row * a.d, a.d, a.eps, red);
}

// ------------------------------------------------------------------ K-slice sums
// The row kernels behind a split K are latency: the partial sums have left the caches of the XCDs that wrote them, a round
// trip takes about a microsecond, and a loop over the slices that adds each as it comes makes a chain of them (residual and
// norm of 128 rows of the 32B shape: 12 slices 7.7 us, 5 slices 6.0; q/k/v in 4 slices 5.2).  They load SLICES slices for
// everything a thread holds before they add any; slices past the last one are the last one again, not added.
template <int SLICES, int N, typename Load>
__device__ __forceinline__ void add_slices(f32x4 (&acc)[N], int split, Load load) {
    for (int s0 = 0; s0 < split; s0 += SLICES) {
        f32x4 p[SLICES][N];
#pragma unroll
        for (int k = 0; k < SLICES; ++k)
#pragma unroll
            for (int j = 0; j < N; ++j) p[k][j] = load(s0 + k < split ? s0 + k : split - 1, j);
#pragma unroll
        for (int k = 0; k < SLICES; ++k)
#pragma unroll
            for (int j = 0; j < N; ++j) {
                const f32x4 sum = acc[j] + p[k][j];
                acc[j] = s0 + k < split ? sum : acc[j];
            }
    }
}
// Slices to load at once: all up to 8, equal shares of more, each number with a kernel of its own: the kernel of the next larger
// one loads the last slice again (with their products, 5 slices of the o projection of 33 to 128 rows and 7 of q/k/v take 1 % less
// than with kernels for 6 and 8).
template <typename F>
static void with_slices(int split, F go) {
    const int rounds = (split + 7) / 8;
    switch ((split + rounds - 1) / rounds) {
        case 0:
        case 1: return go(std::integral_constant<int, 1>{});
        case 2: return go(std::integral_constant<int, 2>{});
        case 3: return go(std::integral_constant<int, 3>{});
        case 4: return go(std::integral_constant<int, 4>{});
        case 5: return go(std::integral_constant<int, 5>{});
        case 6: return go(std::integral_constant<int, 6>{});
        case 7: return go(std::integral_constant<int, 7>{});
        default: return go(std::integral_constant<int, 8>{});
    }
}

// ------------------------------------------------------------------ sum K slices + residual (+ RMSNorm)
// x_out[row] = resid[row] (or 0 if resid is null) + sum_s partial[s][row]; with NORM also
// r_out[row] = rmsnorm(x_out[row]) in bf16.  Workgroups of 512 threads, MAXV pieces of four values each: one a row
// where the norm follows (the row stays in registers between the two passes, d <= 4 * 512 * MAXV), else one a piece
// (grid: rows x pieces), so that a few rows keep more compute units busy.
constexpr int RESID_THREADS = 512;

__device__ __forceinline__ float block_sum512(float v, float* red) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    float t = 0.f;
#pragma unroll
    for (int w = 0; w < RESID_THREADS / 64; ++w) t += red[w];
    return t;
}

template <int MAXV, int SLICES, bool NORM>
__global__ __launch_bounds__(RESID_THREADS) void epi_resid_kernel(const float* __restrict__ partial, int split,
                                                                   size_t slice_stride, const float* __restrict__ resid,
                                                                   float* __restrict__ x_out,
                                                                   const bf16_t* __restrict__ ln_w,
                                                                   bf16_t* __restrict__ r_out, int d, float eps,
                                                                   const int* __restrict__ row_live) {
    __shared__ float red[RESID_THREADS / 64];
    const size_t row = blockIdx.x;
    if (row_live && row_live[row] < 0) return;  // padding row
    const int nv = d / 4, first = (NORM ? 0 : blockIdx.y * RESID_THREADS) + threadIdx.x;
    int at[MAXV];   // a thread past the row's end loads its last piece again and stores nothing
    f32x4 v[MAXV];
    u32x2 gain[MAXV];
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
        at[j] = first + j * RESID_THREADS < nv ? first + j * RESID_THREADS : nv - 1;
        v[j] = resid ? reinterpret_cast<const f32x4*>(resid + row * d)[at[j]] : f32x4{0.f, 0.f, 0.f, 0.f};
        if (NORM) gain[j] = reinterpret_cast<const u32x2*>(ln_w)[at[j]];
    }
    const float* p = partial + row * d;
    add_slices<SLICES>(v, split, [&](int sl, int j) { return reinterpret_cast<const f32x4*>(p + sl * slice_stride)[at[j]]; });
    float ss = 0.f;
#pragma unroll
    for (int j = 0; j < MAXV; ++j) {
        if (first + j * RESID_THREADS >= nv) continue;
        reinterpret_cast<f32x4*>(x_out + row * d)[at[j]] = v[j];
        ss += v[j].x * v[j].x + v[j].y * v[j].y + v[j].z * v[j].z + v[j].w * v[j].w;
    }
    if constexpr (NORM) {
        const float inv = rsqrtf(block_sum512(ss, red) / (float)d + eps);
#pragma unroll
        for (int j = 0; j < MAXV; ++j) {
            if (first + j * RESID_THREADS >= nv) continue;
            const u32x2 g = gain[j];
            u32x2 o;
            o.x = pack_bf16x2(v[j].x * inv * __uint_as_float(g.x << 16), v[j].y * inv * __uint_as_float(g.x & 0xffff0000u));
            o.y = pack_bf16x2(v[j].z * inv * __uint_as_float(g.y << 16), v[j].w * inv * __uint_as_float(g.y & 0xffff0000u));
            reinterpret_cast<u32x2*>(r_out + row * d)[at[j]] = o;
        }
    }
}

// ------------------------------------------------------------------ sum K slices + bias + RoPE + KV append
// One token row and a chunk of its work items (grid: row x chunk; TURN: workgroups [0, rows * chunks)).  Work item = four
// consecutive rotate-half pairs (j..j+3, j+hd/2..j+hd/2+3) of one head: two 16-byte loads per K slice.  q goes to q_out[row], k and v to the
// token's slot in the paged pools.
// TURN: v has workgroups of its own behind these, one kv head of 16 rows each.  A page keeps v as [head_dim][16 tokens],
// so 8 rows whose tokens lie side by side in an aligned half of a page are turned over in LDS and written as 16 bytes
// per head_dim index; others go one by one.  Written one by one throughout, the 2-byte stores at a 32-byte stride are a
// third of the kernel's time in large batches: 32B shape, 2048 rows 30 us, turned over 19; 11104 rows 190 and 92 (478 MB,
// 5.2 TB/s).  Small ones are all latency, and the two barriers of the way through LDS add to it: 32B / 7B shape, slices added
// as they came, 32 rows 5.1 / 5.4 us turned over and 4.0 / 4.0 one by one, 128 rows 6.2 / 5.5 and 5.2 / 4.2, 192 rows 7.6 /
// 5.6 and 8.3 / 5.6; loading all slices first takes as much off either.
constexpr int V_ROWS = 16;
constexpr int TURN_ABOVE = 128;   // rows
template <int HD, bool TURN, int SLICES>
__global__ __launch_bounds__(ROW_THREADS) void epi_qkv_kernel(const float* __restrict__ partial, int split,
                                                               size_t slice_stride, const bf16_t* __restrict__ bias,
                                                               const int* __restrict__ tok_pos,
                                                               const int* __restrict__ tok_slot,
                                                               const float2* __restrict__ rope, int max_pos,
                                                               bf16_t* __restrict__ q_out,
                                                               bf16_t* __restrict__ k_pool, bf16_t* __restrict__ v_pool,
                                                               int n_q, int n_kv, int rows, int chunks) {
    constexpr int half = HD / 2, per_head = half / 4;
    const int width = (n_q + 2 * n_kv) * HD;
    __shared__ __align__(16) bf16_t vt[V_ROWS * (HD + 8)];
    __shared__ int vslot[V_ROWS], vany;
    const int n_qk = rows * chunks;
    if (TURN && (int)blockIdx.x >= n_qk) {
        constexpr int ROW = HD + 8, F4 = HD / 4, PASS = ROW_THREADS / F4;   // rows per pass
        const int vb = blockIdx.x - n_qk, g = vb % n_kv, r0 = (vb / n_kv) * V_ROWS;
        const int c = threadIdx.x % F4;
        if (threadIdx.x < 64) {   // wave 0
            const int row = r0 + threadIdx.x;
            const int slot = threadIdx.x < V_ROWS && row < rows && tok_pos[row] >= 0 ? tok_slot[row] : -1;
            if (threadIdx.x < V_ROWS) vslot[threadIdx.x] = slot;
            const bool any = __builtin_amdgcn_ballot_w64(slot >= 0) != 0;
            if (threadIdx.x == 0) vany = any;
        }
        __syncthreads();
        if (!vany) return;   // padding rows only
        const int col = (n_q + n_kv + g) * HD + 4 * c;
        constexpr int NP = V_ROWS / PASS;
        const float* p[NP];
        f32x4 acc[NP];
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int row = r0 + threadIdx.x / F4 + i * PASS;
            p[i] = partial + (size_t)(row < rows ? row : rows - 1) * width + col;
            acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        float b[4] = {0.f, 0.f, 0.f, 0.f};
        if (bias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) b[e] = bf16_to_f32(bias[col + e]);
        }
        add_slices<SLICES>(acc, split, [&](int sl, int i) { return *reinterpret_cast<const f32x4*>(p[i] + sl * slice_stride); });
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int rr = threadIdx.x / F4 + i * PASS;
            f32x4 a = acc[i];
            if (bias) {
#pragma unroll
                for (int e = 0; e < 4; ++e) a[e] += b[e];
            }
            u32x2 w;
            w.x = pack_bf16x2(a.x, a.y);
            w.y = pack_bf16x2(a.z, a.w);
            *reinterpret_cast<u32x2*>(&vt[rr * ROW + 4 * c]) = w;
        }
        __syncthreads();
        if (threadIdx.x >= 2 * HD) return;
        const int e = threadIdx.x >> 1, h8 = (threadIdx.x & 1) * 8;
        const int s0 = vslot[h8];
        bool whole = s0 >= 0 && s0 % 8 == 0;
#pragma unroll
        for (int i = 1; i < 8; ++i) whole = whole && vslot[h8 + i] == s0 + i;
        if (whole) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[i] = (unsigned)vt[(h8 + 2 * i) * ROW + e] | ((unsigned)vt[(h8 + 2 * i + 1) * ROW + e] << 16);
            bf16_t* dst = v_pool + (((size_t)(s0 / LAPS_PAGE) * n_kv + g) * HD + e) * LAPS_PAGE + s0 % LAPS_PAGE;
            *reinterpret_cast<u32x4*>(dst) = w;
        } else {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int s = vslot[h8 + i];
                if (s >= 0) v_pool[(((size_t)(s / LAPS_PAGE) * n_kv + g) * HD + e) * LAPS_PAGE + s % LAPS_PAGE] = vt[(h8 + i) * ROW + e];
            }
        }
        return;
    }
    const size_t row = TURN ? blockIdx.x / chunks : blockIdx.x;
    const int it = (TURN ? blockIdx.x - (int)row * chunks : blockIdx.y) * ROW_THREADS + threadIdx.x;
    if (it >= (n_q + (TURN ? 1 : 2) * n_kv) * per_head) return;
    const int pos = tok_pos[row], slot = tok_slot[row];
    const int head = it / per_head, j = (it % per_head) * 4;
    const int c0 = head * HD + j, c1 = c0 + half;
    if (pos < 0 || slot < 0) {  // padding row: defined q (zero), no cache write, partial sums not read
        if (head < n_q) {
            const u32x2 z = {0u, 0u};
            *reinterpret_cast<u32x2*>(q_out + row * (size_t)(n_q * HD) + c0) = z;
            *reinterpret_cast<u32x2*>(q_out + row * (size_t)(n_q * HD) + c1) = z;
        }
        return;
    }
    // positions past the table are the caller's error; clamp so that the read stays in bounds
    const float2* cs = rope + (size_t)(pos < max_pos ? pos : max_pos - 1) * half + j;
    float2 turn[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) turn[e] = cs[e];
    float bias_a[4] = {0.f, 0.f, 0.f, 0.f}, bias_b[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias) {
#pragma unroll
        for (int e = 0; e < 4; ++e) bias_a[e] = bf16_to_f32(bias[c0 + e]), bias_b[e] = bf16_to_f32(bias[c1 + e]);
    }
    f32x4 ab[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
    const float* p = partial + row * width;
    add_slices<SLICES>(ab, split, [&](int sl, int h) { return *reinterpret_cast<const f32x4*>(p + sl * slice_stride + (h ? c1 : c0)); });
    f32x4 a = ab[0], b = ab[1];
    if (bias) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            a[e] += bias_a[e];
            b[e] += bias_b[e];
        }
    }
    if (TURN || head < n_q + n_kv) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float2 t = turn[e];
            const float ra = a[e] * t.x - b[e] * t.y;
            const float rb = b[e] * t.x + a[e] * t.y;
            a[e] = ra;
            b[e] = rb;
        }
    }
    u32x2 wa, wb;
    wa.x = pack_bf16x2(a.x, a.y);
    wa.y = pack_bf16x2(a.z, a.w);
    wb.x = pack_bf16x2(b.x, b.y);
    wb.y = pack_bf16x2(b.z, b.w);
    if (head < n_q) {
        *reinterpret_cast<u32x2*>(q_out + row * (size_t)(n_q * HD) + c0) = wa;
        *reinterpret_cast<u32x2*>(q_out + row * (size_t)(n_q * HD) + c1) = wb;
    } else if (TURN || head < n_q + n_kv) {
        bf16_t* dst = k_pool + (((size_t)(slot / LAPS_PAGE) * n_kv + (head - n_q)) * LAPS_PAGE + slot % LAPS_PAGE) * HD;
        *reinterpret_cast<u32x2*>(dst + j) = wa;
        *reinterpret_cast<u32x2*>(dst + j + half) = wb;
    } else {
        bf16_t* dst = v_pool + ((size_t)(slot / LAPS_PAGE) * n_kv + (head - n_q - n_kv)) * HD * LAPS_PAGE + slot % LAPS_PAGE;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            dst[(size_t)(j + e) * LAPS_PAGE] = f32_to_bf16(a[e]);
            dst[(size_t)(j + half + e) * LAPS_PAGE] = f32_to_bf16(b[e]);
        }
    }
}

// ------------------------------------------------------------------ sum K slices + SwiGLU
// Packed gate/up columns: block b of 64 columns = gate cols [32b, 32b+32) then up cols [32b, 32b+32).
template <int SLICES>
__global__ __launch_bounds__(ROW_THREADS) void epi_swiglu_kernel(const float* __restrict__ partial, int split,
                                                                  size_t slice_stride, bf16_t* __restrict__ act,
                                                                  int inter, const int* __restrict__ row_live) {
    const size_t row = blockIdx.x;
    const int width = 2 * inter;
    if (row_live && row_live[row] < 0) return;  // padding row
    {
        const int c4 = blockIdx.y * ROW_THREADS + threadIdx.x;
        if (c4 >= inter / 4) return;
        const int c = c4 * 4;
        const int blk = c / 32, in = c % 32;
        const size_t gcol = (size_t)blk * 64 + in;
        f32x4 gu[2] = {{0.f, 0.f, 0.f, 0.f}, {0.f, 0.f, 0.f, 0.f}};
        const float* p = partial + row * width + gcol;
        add_slices<SLICES>(gu, split, [&](int sl, int h) { return *reinterpret_cast<const f32x4*>(p + sl * slice_stride + 32 * h); });
        const f32x4 g = gu[0], u = gu[1];
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = g[e] / (1.f + __expf(-g[e])) * u[e];
        u32x2 w;
        w.x = pack_bf16x2(o.x, o.y);
        w.y = pack_bf16x2(o.z, o.w);
        *reinterpret_cast<u32x2*>(act + row * inter + c) = w;
    }
}

// ------------------------------------------------------------------ gate/up interleave
__global__ void pack_gate_up_kernel(const u32x4* __restrict__ wg, const u32x4* __restrict__ wu, u32x4* __restrict__ dst,
                                    int inter, int row_vecs) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t total = (size_t)2 * inter * row_vecs;
    if (i >= total) return;
    const size_t drow = i / row_vecs, v = i % row_vecs;
    const size_t blk = drow / 64, in = drow % 64;
    const size_t srow = blk * 32 + (in % 32);
    dst[i] = (in < 32 ? wg : wu)[srow * row_vecs + v];
}

// ------------------------------------------------------------------ token-major K/V <-> pools
// One workgroup per (page of a sequence, kv head): 2 * HD threads, each one 16-byte chunk of K and of V.  A page of K is
// copied as it lies; V changes between [token][HD] and [HD][token] through LDS, so that both sides are 16-byte accesses.
// Bound by memory: 18431 tokens of 8 heads x 128, gather + scatter, moved element by element (2-byte accesses, a
// workgroup per token) 166 us a pair at 1.8 TB/s, now 58 us at 5.2 TB/s (a large copy: 4.8 TB/s).
//
// The first work item of sequence s is cu[s] / 16 + 2 s: a sequence of n tokens touches at most n / 16 + 2 pages, so
// the items of different sequences never overlap and no prefix sum is needed; the spare ones return at once.
// Tokens before cu[0] count to the first sequence and tokens past cu[n_seq] to the last one, as in the kernel below.
template <int HD, bool SCATTER>
__global__ __launch_bounds__(2 * HD) void kv_page_kernel(int n_seq, int n_tokens, const int* __restrict__ cu,
                                                          const int* __restrict__ start_pos,
                                                          const int* __restrict__ page_table, int max_pages,
                                                          u32x4* __restrict__ k_tok, u32x4* __restrict__ v_tok,
                                                          u32x4* __restrict__ k_pool, u32x4* __restrict__ v_pool, int n_kv,
                                                          int n_pool_pages) {
    constexpr int CPR = HD / 8;          // 16-byte chunks per token and head
    constexpr int ROW = HD + 8;          // LDS row: the two halves of a page fall on different banks
    __shared__ __align__(16) bf16_t vt[LAPS_PAGE * ROW];
    const int item = blockIdx.x, head = blockIdx.y, tid = threadIdx.x;
    auto first_token = [&](int s) { return s == 0 ? 0 : cu[s]; };
    auto first_item = [&](int s) { return first_token(s) / LAPS_PAGE + 2 * s; };
    int lo = 0, hi = n_seq;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first_item(mid) <= item) lo = mid; else hi = mid;
    }
    // whatever the arrays hold: tokens stay in [0, n_tokens), pages in the table, page ids in the pool
    const int t0 = first_token(lo), t1 = (lo + 1 < n_seq && cu[lo + 1] < n_tokens) ? cu[lo + 1] : n_tokens;
    if (t0 < 0 || t0 >= t1 || item < first_item(lo)) return;
    const long shift = (long)start_pos[lo] - cu[lo];          // position of a token = its index + shift
    const long page_index = ((t0 + shift) >> 4) + (item - first_item(lo));
    const long a = page_index * LAPS_PAGE - shift;            // token at offset 0 of the page, if the sequence has it
    if (a >= t1 || page_index < 0 || page_index >= max_pages) return;
    const int off0 = a < t0 ? (int)(t0 - a) : 0, off1 = t1 - a < LAPS_PAGE ? (int)(t1 - a) : LAPS_PAGE;
    const int page = page_table[(size_t)lo * max_pages + page_index];
    if (page < 0 || page >= n_pool_pages) return;             // unset table entry, or not a page of the pool
    const size_t pool = ((size_t)page * n_kv + head) * (2 * HD);
    const int off = tid / CPR, c = tid % CPR;                 // token-major: token of the page, chunk of the head
    const bool mine = off >= off0 && off < off1;
    const size_t tok = ((size_t)(a + off) * n_kv + head) * CPR + c;   // only used where `mine`
    const int e = tid >> 1, half = tid & 1;                   // pool V: head_dim index, tokens 8 half .. 8 half + 7
    if (SCATTER) {
        if (mine) {
            k_pool[pool + tid] = k_tok[tok];
            *reinterpret_cast<u32x4*>(&vt[off * ROW + 8 * c]) = v_tok[tok];
        }
        __syncthreads();
        if (off0 <= 8 * half && off1 >= 8 * half + 8) {
            u32x4 w;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                w[i] = (unsigned)vt[(8 * half + 2 * i) * ROW + e] | ((unsigned)vt[(8 * half + 2 * i + 1) * ROW + e] << 16);
            v_pool[pool + tid] = w;
        } else {   // the page also holds tokens that are not moved
            bf16_t* dst = reinterpret_cast<bf16_t*>(v_pool + pool + tid);
#pragma unroll
            for (int i = 0; i < 8; ++i)
                if (8 * half + i >= off0 && 8 * half + i < off1) dst[i] = vt[(8 * half + i) * ROW + e];
        }
    } else {
        const u32x4 w = v_pool[pool + tid];
        if (mine) k_tok[tok] = k_pool[pool + tid];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            vt[(8 * half + 2 * i) * ROW + e] = (bf16_t)w[i];
            vt[(8 * half + 2 * i + 1) * ROW + e] = (bf16_t)(w[i] >> 16);
        }
        __syncthreads();
        if (mine) v_tok[tok] = *reinterpret_cast<const u32x4*>(&vt[off * ROW + 8 * c]);
    }
}

// The same for arrays that are not 16-byte aligned, element by element.
template <bool SCATTER>
__global__ void kv_move_kernel(int n_seq, int n_tokens, const int* __restrict__ cu, const int* __restrict__ start_pos,
                               const int* __restrict__ page_table, int max_pages, bf16_t* __restrict__ k_tok,
                               bf16_t* __restrict__ v_tok, bf16_t* __restrict__ k_pool, bf16_t* __restrict__ v_pool,
                               int n_kv, int hd, int n_pool_pages) {
    const int tok = blockIdx.x;
    if (tok >= n_tokens) return;
    int lo = 0, hi = n_seq;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (cu[mid] <= tok) lo = mid; else hi = mid;
    }
    const int pos = start_pos[lo] + (tok - cu[lo]);
    if (pos < 0 || pos / LAPS_PAGE >= max_pages) return;  // outside the table
    const int page = page_table[(size_t)lo * max_pages + pos / LAPS_PAGE], off = pos % LAPS_PAGE;
    if (page < 0 || page >= n_pool_pages) return;  // unset table entry, or not a page of the pool
    for (int i = threadIdx.x; i < n_kv * hd; i += blockDim.x) {
        const int g = i / hd, e = i % hd;
        const size_t kp = (((size_t)page * n_kv + g) * LAPS_PAGE + off) * hd + e;
        const size_t vp = (((size_t)page * n_kv + g) * hd + e) * LAPS_PAGE + off;
        const size_t tp = (size_t)tok * n_kv * hd + i;
        if (SCATTER) {
            k_pool[kp] = k_tok[tp];
            v_pool[vp] = v_tok[tp];
        } else {
            k_tok[tp] = k_pool[kp];
            v_tok[tp] = v_pool[vp];
        }
    }
}

// Staging of a captured bucket, one launch: workgroup 0 writes the batch's metadata, workgroup 1 + r prepares row r.  Every
// row workgroup scans the slots' lengths itself instead of waiting for workgroup 0 (two launches, 4.8 + 9.4 us for 128
// rows; one, 5.9 us; short re-prefill replay 285 -> 280, single turn 161 -> 156), and its input row is on the way meanwhile.
//
// The lengths the caller staged for the first n_real slots are clamped to [0, len_bucket], the other slots are empty, and
// the sequences are packed one after the other (row_start = running sum of the clamped lengths, so the total never
// exceeds the graph's depth * len_bucket rows whatever the caller's arrays hold).
__device__ __forceinline__ int staged_len(const StageArgs& a, int i) {
    int l = i < a.n_real ? a.seq_len[i] : 0;
    l = l > a.len_bucket ? a.len_bucket : l;
    return l < 0 ? 0 : l;
}

// Rows before this thread's run of consecutive slots [lo, hi) and rows in it; sums: ROW_THREADS / 64 ints of LDS.
__device__ __forceinline__ int staged_scan(const StageArgs& a, int lo, int hi, int* mine_out, int* sums) {
    int mine = 0;
    for (int i = lo; i < hi; ++i) mine += staged_len(a, i);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int v = __shfl_up(incl, o, 64);
        if (lane >= o) incl += v;
    }
    if (lane == 63) sums[wave] = incl;
    __syncthreads();
    int before = incl - mine;
    for (int w = 0; w < wave; ++w) before += sums[w];
    *mine_out = mine;
    return before;
}

__global__ __launch_bounds__(ROW_THREADS) void stage_kernel(const StageArgs a) {
    __shared__ int sums[ROW_THREADS / 64];
    __shared__ float red[ROW_THREADS / 64];
    __shared__ int where[3];   // slot of this row, its first row, live
    const int t = threadIdx.x, depth = a.depth;
    const int per = (depth + ROW_THREADS - 1) / ROW_THREADS;
    const int lo = t * per, hi = (lo + per < depth) ? lo + per : depth;
    int mine;
    if (blockIdx.x == 0) {
        int run = staged_scan(a, lo, hi, &mine, sums);
        for (int i = lo; i < hi; ++i) {
            const int l = staged_len(a, i);
            a.row_start_out[i] = run;
            a.seq_len_out[i] = l;
            a.new_len_out[i] = l;
            const int pf = i < a.n_real ? a.prefix_len[i] : 0;
            a.prefix_out[i] = pf < 0 ? 0 : pf;
            run += l;
        }
        if (t == ROW_THREADS - 1) a.row_start_out[depth] = run;
        __syncthreads();   // the lengths written above are read below by other threads of this workgroup
        laps_dev_attn_sched(a.new_len_out, depth, a.group, a.rows_per_wg, a.tile_start, a.item_seq, a.max_items, sums);
        laps_dev_attn_desc(a.new_len_out, a.prefix_out, a.row_start_out, depth, a.group, a.rows_per_wg, a.max_pages, a.tile_start,
                           a.item_seq, a.max_items, a.n_split, a.min_tiles, a.attn_desc);
        if (a.attn_wgs > 0)
            laps_dev_attn_bounds(a.new_len_out, a.prefix_out, depth, a.group, a.n_kv, a.max_pages, a.tile_start, a.item_seq,
                                 a.max_items, a.attn_wgs, a.attn_pre, a.attn_bounds, sums);
        return;
    }
    const int row = blockIdx.x - 1, n_rows = gridDim.x - 1;
    const f32x4* src = reinterpret_cast<const f32x4*>(a.x_in + (size_t)row * a.d);
    f32x4* copy_to = nullptr;
    if (a.x_rows != nullptr && row < a.n_rows) {
        copy_to = reinterpret_cast<f32x4*>(a.x_in + (size_t)row * a.d);
        src = reinterpret_cast<const f32x4*>(a.x_rows + (size_t)row * a.d);
        if (src == copy_to) copy_to = nullptr;
    }
    RowRegs<ROW_MAXV> r;
    r.load(src, a.ln_w, a.d);
    if (t == 0) where[2] = 0;
    int run = staged_scan(a, lo, hi, &mine, sums);   // its barrier orders the line above before the lines below
    if (row >= run && row < run + mine)
        for (int i = lo; i < hi; ++i) {
            const int l = staged_len(a, i);
            if (row < run + l) {
                where[0] = i;
                where[1] = run;
                where[2] = 1;
                break;
            }
            run += l;
        }
    {   // this workgroup's share of the page-table copy
        const int total = depth * a.max_pages, n_src = a.n_real * a.max_pages;
        const int chunk = (total + n_rows - 1) / n_rows;
        const int end = (row + 1) * chunk < total ? (row + 1) * chunk : total;
        for (int i = row * chunk + t; i < end; i += ROW_THREADS) a.page_table_out[i] = i < n_src ? a.page_table[i] : 0;
    }
    __syncthreads();
    const bool live = where[2] != 0;
    if (t == 0) {   // token position and cache slot, as in token_meta; page ids from the caller's table
        int pos = -1, slot = -1;
        if (live) {
            const int s = where[0], h = a.prefix_len[s];
            pos = (h > 0 ? h : 0) + row - where[1];
            const int pi = pos / LAPS_PAGE;
            const int page = pi < a.max_pages ? a.page_table[(size_t)s * a.max_pages + pi] : -1;
            slot = (page >= 0 && page < a.n_pool_pages) ? page * LAPS_PAGE + pos % LAPS_PAGE : -1;
        }
        a.tok_pos[row] = pos;
        a.tok_slot[row] = slot;
    }
    if (copy_to) r.store(copy_to, a.d);
    if (!live) return;   // padding row: nothing reads its normed row
    r.norm(a.r0 + (size_t)row * a.d, a.d, a.eps, red);
}

}  // namespace

int laps_launch_stage(const StageArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(stage_kernel, dim3(a.depth * a.len_bucket + 1), dim3(ROW_THREADS), 0, s, a);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_rope_table(float2* table, int max_pos, int head_dim, float theta, hipStream_t s) {
    const int half = head_dim / 2;
    const int n = max_pos * half;
    hipLaunchKernelGGL(rope_table_kernel, dim3((n + 255) / 256), dim3(256), 0, s, table, max_pos, half, (double)theta,
                       head_dim);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_begin(const BeginArgs& a, hipStream_t s) {
    auto kern = a.d <= 4 * ROW_THREADS ? begin_kernel<1> : begin_kernel<ROW_MAXV>;   // d <= 8192 (check_cfg)
    hipLaunchKernelGGL(kern, dim3(1 + a.n_rows), dim3(ROW_THREADS), 0, s, a);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_rmsnorm(const float* x, const bf16_t* w, bf16_t* out, int rows, int d, float eps, const int* row_live,
                        hipStream_t s) {
    auto kern = d <= 4 * ROW_THREADS ? rmsnorm_kernel<1> : rmsnorm_kernel<ROW_MAXV>;   // d <= 8192 (check_cfg)
    hipLaunchKernelGGL(kern, dim3(rows), dim3(ROW_THREADS), 0, s, x, w, out, d, eps, row_live);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_epi_resid(const float* partial, int split, const float* resid, float* x_out, const bf16_t* ln_w,
                          bf16_t* r_out, int rows, int d, float eps, const int* row_live, hipStream_t s) {
    const size_t stride = (size_t)rows * d;
    const int pieces = (d / 4 + RESID_THREADS - 1) / RESID_THREADS;
    if (pieces > 4) {
        laps_set_error("row width %d too large for the fused residual + norm kernel (max %d)", d, 4 * RESID_THREADS * 4);
        return LAPS_EINVAL;
    }
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(rows, ln_w ? 1 : pieces), dim3(RESID_THREADS), 0, s, partial, split, stride, resid, x_out,
                           ln_w, r_out, d, eps, row_live);
    };
    with_slices(split, [&](auto slices) {
        constexpr int S = decltype(slices)::value;
        if (!ln_w) go(epi_resid_kernel<1, S, false>);
        else if (pieces == 1) go(epi_resid_kernel<1, S, true>);
        else if (pieces == 2) go(epi_resid_kernel<2, S, true>);
        else if (pieces == 3) go(epi_resid_kernel<3, S, true>);
        else go(epi_resid_kernel<4, S, true>);
    });
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_epi_qkv(const float* partial, int split, const bf16_t* bias, const int* tok_pos, const int* tok_slot,
                        const float2* rope, int max_pos, bf16_t* q_out, bf16_t* k_pool, bf16_t* v_pool, int rows,
                        int n_q, int n_kv, int hd, hipStream_t s) {
    const size_t stride = (size_t)rows * (n_q + 2 * n_kv) * hd;
    const bool turn = rows > TURN_ABOVE;
    const int chunks = ((n_q + (turn ? 1 : 2) * n_kv) * (hd / 8) + ROW_THREADS - 1) / ROW_THREADS;
    const dim3 grid = turn ? dim3(rows * chunks + (rows + V_ROWS - 1) / V_ROWS * n_kv) : dim3(rows, chunks);
    with_slices(split, [&](auto slices) {   // head_dim is one of the two (check_cfg)
        constexpr int S = decltype(slices)::value;
        auto kern = turn ? (hd == 128 ? epi_qkv_kernel<128, true, S> : epi_qkv_kernel<64, true, S>)
                         : (hd == 128 ? epi_qkv_kernel<128, false, S> : epi_qkv_kernel<64, false, S>);
        hipLaunchKernelGGL(kern, grid, dim3(ROW_THREADS), 0, s, partial, split, stride, bias, tok_pos, tok_slot, rope,
                           max_pos, q_out, k_pool, v_pool, n_q, n_kv, rows, chunks);
    });
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_epi_swiglu(const float* partial, int split, bf16_t* act, int rows, int inter, const int* row_live,
                           hipStream_t s) {
    const size_t stride = (size_t)rows * 2 * inter;
    with_slices(split, [&](auto slices) {
        constexpr int S = decltype(slices)::value;
        hipLaunchKernelGGL(epi_swiglu_kernel<S>, dim3(rows, (inter / 4 + ROW_THREADS - 1) / ROW_THREADS), dim3(ROW_THREADS), 0, s, partial,
                           split, stride, act, inter, row_live);
    });
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_pack_gate_up(const bf16_t* wg, const bf16_t* wu, bf16_t* dst, int inter, int d, hipStream_t s) {
    const int row_vecs = d / 8;
    const size_t total = (size_t)2 * inter * row_vecs;
    hipLaunchKernelGGL(pack_gate_up_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s,
                       reinterpret_cast<const u32x4*>(wg), reinterpret_cast<const u32x4*>(wu),
                       reinterpret_cast<u32x4*>(dst), inter, row_vecs);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

int laps_launch_kv_move(bool scatter, int n_seq, int n_tokens, const int* cu, const int* start_pos,
                        const int* page_table, int max_pages, bf16_t* k_tok, bf16_t* v_tok, bf16_t* k_pool,
                        bf16_t* v_pool, int n_kv, int hd, int n_pool_pages, hipStream_t s) {
    if (n_tokens == 0) return LAPS_OK;
    const uintptr_t any = (uintptr_t)k_tok | (uintptr_t)v_tok | (uintptr_t)k_pool | (uintptr_t)v_pool;
    if (any % 16 == 0 && (hd == 64 || hd == 128)) {
        const dim3 grid(n_tokens / LAPS_PAGE + 2 * n_seq, n_kv);
        auto kern = hd == 128 ? (scatter ? kv_page_kernel<128, true> : kv_page_kernel<128, false>)
                              : (scatter ? kv_page_kernel<64, true> : kv_page_kernel<64, false>);
        hipLaunchKernelGGL(kern, grid, dim3(2 * hd), 0, s, n_seq, n_tokens, cu, start_pos, page_table, max_pages,
                           reinterpret_cast<u32x4*>(k_tok), reinterpret_cast<u32x4*>(v_tok),
                           reinterpret_cast<u32x4*>(k_pool), reinterpret_cast<u32x4*>(v_pool), n_kv, n_pool_pages);
    } else if (scatter)
        hipLaunchKernelGGL(kv_move_kernel<true>, dim3(n_tokens), dim3(256), 0, s, n_seq, n_tokens, cu, start_pos,
                           page_table, max_pages, k_tok, v_tok, k_pool, v_pool, n_kv, hd, n_pool_pages);
    else
        hipLaunchKernelGGL(kv_move_kernel<false>, dim3(n_tokens), dim3(256), 0, s, n_seq, n_tokens, cu, start_pos,
                           page_table, max_pages, k_tok, v_tok, k_pool, v_pool, n_kv, hd, n_pool_pages);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}
