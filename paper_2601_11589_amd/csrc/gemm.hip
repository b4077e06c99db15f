// bf16 x bf16 -> fp32 GEMM on gfx950 MFMA, LDS-staged tiles.
//
//   C[M,N] = A[M,K] * W[N,K]^T        A: activations (row-major, K contiguous)
//                                      W: weights in [out, in] order (row-major, K contiguous)
//
// Both operands are K-contiguous, so a lane's MFMA fragment (8 consecutive k of one row) is one
// 16-byte read.  A workgroup owns a BM x BN output tile and one K slice, and walks it in slabs of 64.
//
// Two kinds of tile:
//  * dma_tile (v_mfma_f32_16x16x32_bf16): slabs go straight into LDS; operands of 16-byte alignment and rows of less than
//    2^22 values;
//  * far_tile (v_mfma_f32_32x32x16_bf16): slabs go HBM -> registers -> LDS, every row has a pointer; the longer rows, which
//    32-bit offsets do not reach, and operands that are aligned to their elements only.
//
// far_tile's K loop is software-pipelined by hand:
//   * fragments of k-step kk+1 are read from LDS into a second register set before the MFMAs of
//     k-step kk are issued, so LDS latency hides behind the MFMAs;
//   * the registers holding slab kt+1 are written to the other LDS buffer in the middle of slab kt
//     and immediately reloaded from HBM with slab kt+1+WS; WS = 2 sets of staging registers keep two
//     slabs in flight;
//   * the one barrier per slab sits in the middle of the last k-step's MFMAs and waits on LDS
//     traffic only, never on the HBM loads in flight.
// Epilogues: raw K-slice partial sums (split-K, reduced deterministically by the row kernels in
// elementwise.hip), residual add (fp32 out), or SwiGLU on interleaved gate/up columns (bf16 out).
//
// Workgroup ids are remapped so that each of the 8 XCDs (workgroups are dealt to them round-robin)
// gets a contiguous range of tiles, walked M-fastest in groups of 8 row tiles: the workgroups
// sharing a weight panel sit on one XCD and hit its L2.
#include <algorithm>
#include <type_traits>

#include "laps_internal.h"

namespace {

constexpr int BK = 64;          // k elements per slab: 128 bytes per tile row
constexpr int CHUNKS = BK / 8;  // 16-byte chunks per tile row
constexpr int NUM_XCD = 8;
constexpr int GROUP_M = 8;

// Tile rows are 128 bytes; chunk c of row r is stored at chunk position c ^ f(r).  f makes any 8
// consecutive rows hit 8 different 16-byte columns and any 16 consecutive rows hit 16 different
// 16-byte columns of a 256-byte bank line, for both fragment reads (lanes = consecutive rows, same
// chunk) and slab writes (8 lanes = one row, all chunks).
__device__ __forceinline__ int swz(int row, int chunk) { return chunk ^ ((row & 7) ^ ((row >> 3) & 1)); }

// LDS-only barrier: waits for this wave's LDS reads/writes, not for global loads in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

template <int BM, int BN, int WM, int WN>
struct Traits {
    static constexpr int NT = WM * WN * 64;
    static constexpr int WTM = BM / WM, WTN = BN / WN;
    static constexpr int MI = WTM / 32, NI = WTN / 32;
    static constexpr int A_LOADS = BM * CHUNKS / NT, B_LOADS = BN * CHUNKS / NT;
    static constexpr int LDS_BYTES = 2 * (BM + BN) * BK * 2;
    // 4-wave workgroups small enough for two of them on a compute unit get the registers for it (two waves per SIMD):
    // one's epilogue and barriers then hide under the other's products
    static constexpr int WAVES_PER_SIMD = (NT == 256 && 2 * LDS_BYTES <= 160 * 1024) ? 2 : 1;
    static_assert(BM * CHUNKS % NT == 0 && BN * CHUNKS % NT == 0, "tile rows must divide over threads");
    static_assert(WTM % 32 == 0 && WTN % 32 == 0, "wave tile must be a multiple of the 32x32 MFMA");
};

// 16-byte accesses to the caller's arrays, which are aligned to their elements only
typedef f32x4 f32x4_a4 __attribute__((aligned(4)));
typedef u32x4 u32x4_a2 __attribute__((aligned(2)));

struct TileCoord {
    int tm, tn, ks;
};

// x / d of a uniform x >= 0: one reciprocal and a correction (the compiler's own division is several times as long, and
// four of them stood in front of every workgroup's first load).  The quotient is off by one at most below 2^23.
__device__ __forceinline__ int fast_div(int x, int d) {
    const int q = (int)((float)x * __builtin_amdgcn_rcpf((float)d));
    const int r = x - q * d;
    return __builtin_amdgcn_readfirstlane(q + (r >= d ? 1 : 0) - (r < 0 ? 1 : 0));
}

__device__ __forceinline__ TileCoord map_block(int bid, int tiles_m, int tiles_n, int split) {
    const int total = tiles_m * tiles_n * split;
    const int xcd = bid % NUM_XCD, idx = bid / NUM_XCD;
    const int q = total / NUM_XCD, r = total % NUM_XCD;
    const int lin = xcd * q + (xcd < r ? xcd : r) + idx;  // contiguous range per XCD
    const int per_split = tiles_m * tiles_n;
    TileCoord c;
    c.ks = split == 1 ? 0 : fast_div(lin, per_split);
    const int t = lin - c.ks * per_split;
    if (tiles_m == 1) {
        c.tm = 0;
        c.tn = t;
        return c;
    }
    const int gsize = GROUP_M * tiles_n;
    const int grp = fast_div(t, gsize);
    const int first_m = grp * GROUP_M;
    const int gm = (tiles_m - first_m) < GROUP_M ? (tiles_m - first_m) : GROUP_M;
    const int in = t - grp * gsize;
    c.tn = fast_div(in, gm);
    c.tm = first_m + in - c.tn * gm;
    return c;
}

struct GemmArgs {
    const bf16_t* A;
    const bf16_t* W;
    int M, N, K, split, kps, tiles_m, tiles_n;
    float* out_f32;        // EPI_PARTIAL: [split][M][N]; EPI_RESID: [M][N]
    const float* resid;    // EPI_RESID: [M][N] (may alias out_f32)
    bf16_t* out_bf16;      // EPI_SWIGLU: [M][N/2]
    const int* row_live;   // [M] or NULL: rows with a negative entry are padding - a row tile that holds nothing else is
                           // skipped (its output is then not written), and dma_tile loads none of them
    const int* n_live;     // NULL, or where the number of leading rows that are not padding is found (at most M count)
    int cols;              // columns of W and of the output that the tiles cover; N apart from them is the outputs' row length
};

// Writes a workgroup's accumulators with the requested epilogue.  Accumulator layout of the 32x32 MFMA:
// lane -> column (lane & 31); register r -> row 8*(r/4) + 4*(lane/32) + r%4.
template <typename T, int EPI>
__device__ __forceinline__ void store_tile(const f32x16 (&acc)[T::MI][T::NI], const GemmArgs& g, int M, int ks, int m0,
                                           int n0, int wm, int wn, int lrow, int lk) {
    const int N = g.N;   // M: rows to store
    if constexpr (EPI == EPI_PARTIAL) {
        float* out = g.out_f32 + (size_t)ks * g.M * N;
#pragma unroll
        for (int mi = 0; mi < T::MI; ++mi)
#pragma unroll
            for (int ni = 0; ni < T::NI; ++ni) {
                const int n = n0 + wn * T::WTN + ni * 32 + lrow;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = m0 + wm * T::WTM + mi * 32 + 8 * (r / 4) + 4 * lk + (r % 4);
                    if (m < M) out[(size_t)m * N + n] = acc[mi][ni][r];
                }
            }
    } else if constexpr (EPI == EPI_RESID) {
        // resid may be the output array itself (every element is read by the thread that writes it), so the compiler
        // keeps a load behind every store before it; written element by element, a lane's 80..256 results take as many
        // memory round trips one after the other (45-70 us per launch whatever the size).  The residual of sub-tile
        // i + 1 is therefore loaded before sub-tile i is stored: one round trip per sub-tile of 16, overlapped.
        // o projection of the 32B layer, 2048 rows, when it ran on these tiles: 165 -> 102 us; a 227 x 256 x 256 product: 45 -> 15.
        constexpr int NS = T::MI * T::NI;
        float rbuf[2][16];
        auto row = [&](int i, int r) { return m0 + wm * T::WTM + (i / T::NI) * 32 + 8 * (r / 4) + 4 * lk + (r % 4); };
        auto col = [&](int i) { return n0 + wn * T::WTN + (i % T::NI) * 32 + lrow; };
        auto load = [&](int i) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = row(i, r);
                rbuf[i & 1][r] = g.resid[(size_t)(m < M ? m : M - 1) * N + col(i)];
            }
        };
        load(0);
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            if (i + 1 < NS) load(i + 1);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = row(i, r);
                if (m < M) g.out_f32[(size_t)m * N + col(i)] = rbuf[i & 1][r] + acc[i / T::NI][i % T::NI][r];
            }
        }
    } else {  // EPI_SWIGLU: sub-tile 2j holds gate columns, sub-tile 2j+1 the matching up columns
        static_assert(EPI != EPI_SWIGLU || T::NI % 2 == 0, "SwiGLU epilogue pairs 32-column sub-tiles");
        const int half_n = N / 2;
#pragma unroll
        for (int mi = 0; mi < T::MI; ++mi)
#pragma unroll
            for (int j = 0; j < T::NI / 2; ++j) {
                const int col = (n0 + wn * T::WTN) / 2 + j * 32 + lrow;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int m = m0 + wm * T::WTM + mi * 32 + 8 * (r / 4) + 4 * lk + (r % 4);
                    if (m < M) {
                        const float gt = acc[mi][2 * j][r], up = acc[mi][2 * j + 1][r];
                        g.out_bf16[(size_t)m * half_n + col] = f32_to_bf16(gt / (1.f + __expf(-gt)) * up);
                    }
                }
            }
    }
}

// The 32-bit offsets of buffer descriptors hold a tile of 320 rows up to K = 2^22 (dma_tile); longer rows take tiles that
// address every row by a pointer.
constexpr int kMaxBufferK = 1 << 22;

// WS = number of register sets that stage slabs: WS slabs (A and W chunks alike - loads return in
// issue order, so a shallower A stream would throttle the W stream) are in flight per workgroup.
// With WS = 2 the K loop is unrolled so that every set index is static, and a K slice must hold a multiple of
// two slabs; WS = 1 serves K of an odd number of slabs (and 192x128, whose second set costs the second workgroup's
// registers).
//
// One tile of the rows_in live rows: workgroup `bid` of tiles_m * tiles_n * g.split.
template <int BM, int BN, int WM, int WN, int EPI, int WS>
__device__ __forceinline__ void far_tile(const GemmArgs& g, unsigned char* smem, const int M, const int tiles_m,
                                         const int tiles_n, const int bid) {
    using T = Traits<BM, BN, WM, WN>;
    u32x4* As = reinterpret_cast<u32x4*>(smem);  // [2][BM][CHUNKS]
    u32x4* Bs = As + 2 * BM * CHUNKS;            // [2][BN][CHUNKS]

    const int K = g.K;
    const TileCoord tc = map_block(bid, tiles_m, tiles_n, g.split);
    const int m0 = tc.tm * BM, n0 = tc.tn * BN;
    const int kbeg = tc.ks * g.kps;
    const int kend = (kbeg + g.kps < K) ? (kbeg + g.kps) : K;
    const int KT = (kend - kbeg) / BK;

    const int tid = threadIdx.x;
    if (g.row_live != nullptr) {  // a row tile made of padding only has nothing to compute (and nothing reads its output)
        bool any = false;
        for (int r = tid; r < BM; r += T::NT) any |= (m0 + r < M) && g.row_live[m0 + r] >= 0;
        // in the slab buffers, not in LDS of its own: two 192x128 workgroups take exactly a unit's 160 KB
        int* flag = reinterpret_cast<int*>(smem);
        const bool wave_any = __builtin_amdgcn_ballot_w64(any) != 0;
        if ((tid & 63) == 0) flag[tid >> 6] = wave_any;
        __syncthreads();
        int live = 0;
#pragma unroll
        for (int w = 0; w < T::NT / 64; ++w) live |= flag[w];
        if (!live) return;
        __syncthreads();   // the flags are read before the first slab overwrites them
    }
    const int lane = tid & 63, wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int lrow = lane & 31, lk = lane >> 5;

    // Slab copy assignment: 16-byte chunk c = tid + i*NT -> row c / CHUNKS = row0 + i * RPP, chunk kc.  RPP is a multiple
    // of 16, so all rows of a thread share one swizzle and their LDS places differ by a constant.
    constexpr int RPP = T::NT / CHUNKS;
    static_assert(RPP % 16 == 0, "rows of a thread must share a swizzle");
    const int row0 = tid / CHUNKS, kc0 = tid % CHUNKS;
    const int dst0 = row0 * CHUNKS + swz(row0, kc0);
    const u32x4_a2* ag[T::A_LOADS];
    const u32x4_a2* bg[T::B_LOADS];
    u32x4 rrb[WS][T::B_LOADS];   // staged W slabs: slab j lives in set j % WS
#pragma unroll
    for (int i = 0; i < T::B_LOADS; ++i) {
        bg[i] = reinterpret_cast<const u32x4_a2*>(g.W + (size_t)(n0 + row0 + i * RPP) * K + kbeg) + kc0;
        rrb[0][i] = *bg[i];
    }
    u32x4 rra[WS][T::A_LOADS];   // staged A slabs, same rule as rrb
#pragma unroll
    for (int i = 0; i < T::A_LOADS; ++i) {
        const int row = row0 + i * RPP;
        const int gr = (m0 + row < M) ? (m0 + row) : (M - 1);  // clamp: rows past M are never stored
        ag[i] = reinterpret_cast<const u32x4_a2*>(g.A + (size_t)gr * K + kbeg) + kc0;
    }
    // fragment read offsets (in 16-byte chunks) inside one LDS buffer, per k-step
    int a_src[T::MI], b_src[T::NI];
#pragma unroll
    for (int mi = 0; mi < T::MI; ++mi) a_src[mi] = (wm * T::WTM + mi * 32 + lrow) * CHUNKS;
#pragma unroll
    for (int ni = 0; ni < T::NI; ++ni) b_src[ni] = (wn * T::WTN + ni * 32 + lrow) * CHUNKS;
    const int a_sw = (lrow & 7) ^ ((lrow >> 3) & 1);  // rows differ by multiples of 32: same swizzle key

    f32x16 acc[T::MI][T::NI];
#pragma unroll
    for (int mi = 0; mi < T::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < T::NI; ++ni)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[mi][ni][r] = 0.f;

    bf16x8 fa[2][T::MI], fb[2][T::NI];
    constexpr int NM = T::MI * T::NI;            // MFMAs per k-step
    constexpr int NF = T::MI + T::NI;            // fragment reads per k-step
    constexpr int NC = T::A_LOADS + T::B_LOADS;  // slab copy operations (global load + LDS store pairs)
    constexpr int NC0 = (NC + 1) / 2;            // copies handled in k-step 0; the rest in k-step 1

    auto clampk = [&](int kt) { return kt < KT ? kt : KT - 1; };  // tail: reload a valid slab, never used
    // copy op i of the slab pipeline: i < A_LOADS moves an A chunk, else a W chunk held in set `ws`
    auto gload_one = [&](int i, int kt, int ws) {
        const int j = i - T::A_LOADS;
        if (i < T::A_LOADS) rra[ws][i] = ag[i][clampk(kt) * CHUNKS];
        else rrb[ws][j] = bg[j][clampk(kt) * CHUNKS];
    };
    auto lstore_one = [&](int i, int buf, int ws) {
        if (i < T::A_LOADS) As[buf * BM * CHUNKS + dst0 + i * RPP * CHUNKS] = rra[ws][i];
        else Bs[buf * BN * CHUNKS + dst0 + (i - T::A_LOADS) * RPP * CHUNKS] = rrb[ws][i - T::A_LOADS];
    };
    // order of need by the MFMA sequence (mi-major): A row block 0, every B column block, remaining A
    auto fload_one = [&](int i, int buf, int kk, int set) {
        const int ch = (kk * 2 + lk) ^ a_sw;
        if (i == 0) fa[set][0] = __builtin_bit_cast(bf16x8, As[buf * BM * CHUNKS + a_src[0] + ch]);
        else if (i <= T::NI) fb[set][i - 1] = __builtin_bit_cast(bf16x8, Bs[buf * BN * CHUNKS + b_src[i - 1] + ch]);
        else fa[set][i - T::NI] = __builtin_bit_cast(bf16x8, As[buf * BM * CHUNKS + a_src[i - T::NI] + ch]);
    };
    auto mma_one = [&](int i, int set) {
        const int mi = i / T::NI, ni = i % T::NI;
        acc[mi][ni] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][mi], fb[set][ni], acc[mi][ni], 0, 0, 0);
    };

    // prologue: slab 0 through the registers into LDS buffer 0 (its W part is on its way), then slabs 1..WS in flight
#pragma unroll
    for (int i = 0; i < T::A_LOADS; ++i) gload_one(i, 0, 0);
#pragma unroll
    for (int i = 0; i < NC; ++i) lstore_one(i, 0, 0);
#pragma unroll
    for (int w = 1; w <= WS; ++w)
#pragma unroll
        for (int i = 0; i < NC; ++i) gload_one(i, w, w % WS);
    lds_barrier();
#pragma unroll
    for (int i = 0; i < NF; ++i) fload_one(i, 0, 0, 0);

    // One memory operation is slotted behind each MFMA so that the matrix pipe never waits for a
    // clump of LDS / HBM instructions to issue (one wave per SIMD: nothing else would feed it).
    //   k-step 0: MFMAs on set 0 | reads of k-step 1 fragments -> set 1 | first half of the slab copy
    //   k-step 1: MFMAs on set 1 | reads of k-step 2 fragments -> set 0 | second half of the slab copy
    //   k-step 2: MFMAs on set 0 | reads of k-step 3 fragments -> set 1
    //   k-step 3: MFMAs on set 1 | barrier half way | reads of the next slab's k-step 0 -> set 0
    // A slab copy = store the staged slab kt+1 to the other LDS buffer, then reload the set just freed
    // with slab kt+1+WS from HBM.  The tail iterations keep the same
    // instruction stream (no branches in the pipeline): they re-store and re-load the last slab, which
    // nothing reads afterwards.
    for (int kt0 = 0; kt0 < KT; kt0 += WS) {
#pragma unroll
        for (int u = 0; u < WS; ++u) {
            const int kt = kt0 + u;
            const int cur = (WS == 1) ? (kt & 1) : (u & 1);  // WS is 1 or even
            const int ws = (u + 1) % WS;                     // set holding W slab kt+1
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                mma_one(i, 0);
#pragma unroll
                for (int o = i; o < NF + NC0; o += NM) {
                    if (o < NF) fload_one(o, cur, 1, 1);
                    else {
                        lstore_one(o - NF, cur ^ 1, ws);
                        gload_one(o - NF, kt + 1 + WS, ws);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                mma_one(i, 1);
#pragma unroll
                for (int o = i; o < NF + (NC - NC0); o += NM) {
                    if (o < NF) fload_one(o, cur, 2, 0);
                    else {
                        lstore_one(NC0 + o - NF, cur ^ 1, ws);
                        gload_one(NC0 + o - NF, kt + 1 + WS, ws);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int i = 0; i < NM; ++i) {
                mma_one(i, 0);
#pragma unroll
                for (int o = i; o < NF; o += NM) fload_one(o, cur, 3, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            constexpr int NH = NM / 2;
#pragma unroll
            for (int i = 0; i < NH; ++i) mma_one(i, 1);
            __builtin_amdgcn_sched_barrier(0);
            lds_barrier();
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = NH; i < NM; ++i) {
                mma_one(i, 1);
#pragma unroll
                for (int o = i - NH; o < NF; o += NM - NH) fload_one(o, cur ^ 1, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }

    store_tile<T, EPI>(acc, g, M, tc.ks, m0, n0, wm, wn, lrow, lk);
}

// ------------------------------------------------------------------ slabs straight into LDS
// What bounds the tiles of 192 and more rows on real data is power: the same kernel runs 1.15 times as fast on zeros.
// Measured on normal(0, 1) x normal(0, 0.02) operands:
//  * v_mfma_f32_16x16x32_bf16 draws less than v_mfma_f32_32x32x16_bf16 (half the accumulator traffic per flop): 2.0-2.1
//    against 1.76-1.85 PFLOP/s with registers alone;
//  * slabs written into LDS by the load instruction itself, without staging registers and LDS stores;
//  * a fragment held for several matrix instructions, and only one operand changed from each to the next (1 %).
// Up to 128 rows the weights' stream bounds, and the loads that bypass the registers can bypass the caches as well.
// 2048 x 55296 x 5120 with SwiGLU: 925 us through registers with 32x32x16, 865 with 16x16x32, 832 this way; 2048 x 5120 x
// 27648: 500, 465, 445; 700 x 27648 x 5120: 204, 192, 180.  Up to 128 rows, weights cold, through registers and this way: 32B
// gate/up at 64 / 128 rows 98 -> 92 / 110 -> 104, q/k/v in 4 slices at 8 / 64 / 128 rows 15.7 -> 13.4 / 19.3 -> 16.4 / 22.0 ->
// 21.0, o in 5 at 8 / 96 rows 12.3 -> 10.6 / 16.7 -> 15.5, down in 12 at 64 / 128 rows 51.5 -> 47.9 / 58.9 -> 54.
// Slabs go in half slabs - the rows that one half of every wave's tile needs of A, and one half of B - through a ring of NS
// of them (2.5 slabs on 256 x 256, the unit's 160 KB of LDS).  All fragments of a half slab (both k-steps of 32) are in
// registers before its products begin, so its place in the ring is free half a slab after it was waited for.
template <int BM, int BN, int WM, int WN>
struct DmaTraits {
    static constexpr int WTM = BM / WM, WTN = BN / WN;                   // wave tile
    static constexpr int MI = WTM / 16, NI = WTN / 16;
    static constexpr int HA = BM / 2, HB = BN / 2;                       // rows of a half slab
    static constexpr int QA = HA / 4, QB = HB / 4;                       // rows that one wave loads
    static constexpr int LA = (QA + 7) / 8, LB = (QB + 7) / 8;           // load instructions of a wave: 8 rows of 128 bytes
    static constexpr int LOADS = LA + LB;
    static constexpr int SLOT = (HA + HB) * BK * 2;                      // bytes
    static constexpr bool TWO = BM * BN <= 192 * 128;                    // two workgroups on a compute unit
    // One workgroup per unit: accumulators in the half of the registers that only matrix instructions compute in, and past
    // that half (320 x 256) in the other.
    static constexpr __host__ __device__ bool in_vgpr(int mi, int ni) { return TWO || mi * NI + ni >= 64; }
    static constexpr int CAP = (TWO ? 80 : 160) * 1024;
    static constexpr int NS = CAP / SLOT < 6 ? CAP / SLOT : 6;           // half slabs in LDS
    static constexpr int LDS = NS * SLOT;
    // The last column tile may reach past N.  Not on 320 x 256, whose offsets of B lie partly in the scalar offset, which the
    // descriptor's bound does not see.
    static constexpr bool RAGGED = BM <= 256;
    static_assert(WM * WN == 4 && QA % 8 == 0 && QB % 4 == 0, "four waves load whole groups of rows");
    static_assert((WTM / 2) % 16 == 0 && (WTN / 2) % 16 == 0, "halves of whole sub-tiles");
    static_assert((WTM / 2) % QA == 0 && (WTN / 2) % QB == 0, "the rows that a wave loads lie in one wave tile");
};

// LDS rows are 128 bytes; chunk c of row r is stored at chunk position c ^ key.  The 16 rows of a fragment have, two by
// two, 8 different keys, so the 16 lanes that read the same chunk of them hit 16 different 16-byte columns of a 256-byte
// bank line (SQ_LDS_BANK_CONFLICT reads 0).  Fragment row i of sub-tile s is row 16 s + i, or with PAIRED columns
// 32 (s / 2) + 8 (i / 4) + 4 (s % 2) + i % 4.
template <bool PAIRED>
__device__ __forceinline__ int dma_key(int row) { return PAIRED ? ((row >> 1) & 1) | (((row >> 3) & 3) << 1) : (row >> 1) & 7; }

typedef __attribute__((ext_vector_type(4))) int i32x4;

// The weights are the matrix instruction's first operand, so that a lane holds four consecutive columns (16 ni + 4 lk + r)
// of row lane & 15 of a sub-tile.
// GUARD: the tile reaches past column N.  (A test in front of every load and store of whole tiles too keeps the loads from
// being issued together: a layer of 227 rows of the tiny model 41.5 -> 44.0 us.)
template <typename D, int EPI, bool GUARD>
__device__ __forceinline__ void store_dma_tile(const f32x4 (&acc)[D::MI][D::NI], const GemmArgs& g, int M, int ks, int m0,
                                               int n0, int wm, int wn, int lrow, int lk) {
    const int N = g.N;
    const int row0 = m0 + wm * D::WTM + lrow, col0 = n0 + wn * D::WTN;
    const auto inside = [&](int ni) { return !GUARD || col0 + ni * 16 < g.cols; };   // wave-uniform; cols is a multiple of 64
    if constexpr (EPI == EPI_PARTIAL) {
        float* out = g.out_f32 + (size_t)ks * g.M * N + col0 + 4 * lk;
#pragma unroll
        for (int mi = 0; mi < D::MI; ++mi) {
            const int m = row0 + mi * 16;
            if (m >= M) continue;
            f32x4_a4* dst = reinterpret_cast<f32x4_a4*>(out + (size_t)m * N);
#pragma unroll
            for (int ni = 0; ni < D::NI; ++ni)
                if (inside(ni)) dst[ni * 4] = acc[mi][ni];
        }
    } else if constexpr (EPI == EPI_RESID) {
        // resid may be the output array itself (every element is read by the thread that writes it), so the compiler
        // keeps a load behind every store before it: the residual of sub-tile row mi + 1 is loaded before row mi is stored.
        // Written element by element, a lane's results took as many memory round trips one after the other (o projection of
        // the 32B layer, 2048 rows: 165 us; ahead: 102).
        f32x4 rbuf[2][D::NI];
        const float* res = g.resid + col0 + 4 * lk;
        float* out = g.out_f32 + col0 + 4 * lk;
        auto load = [&](int mi) {
            const int m = row0 + mi * 16;
            const f32x4_a4* src = reinterpret_cast<const f32x4_a4*>(res + (size_t)(m < M ? m : M - 1) * N);
#pragma unroll
            for (int ni = 0; ni < D::NI; ++ni)
                if (inside(ni)) rbuf[mi & 1][ni] = src[ni * 4];
        };
        load(0);
#pragma unroll
        for (int mi = 0; mi < D::MI; ++mi) {
            if (mi + 1 < D::MI) load(mi + 1);
            const int m = row0 + mi * 16;
            if (m >= M) continue;
            f32x4_a4* dst = reinterpret_cast<f32x4_a4*>(out + (size_t)m * N);
#pragma unroll
            for (int ni = 0; ni < D::NI; ++ni)
                if (inside(ni)) dst[ni * 4] = rbuf[mi & 1][ni] + acc[mi][ni];
        }
    } else {  // EPI_SWIGLU: sub-tiles 4j, 4j+1 hold gate columns, 4j+2, 4j+3 the matching up columns; PAIRED order: a lane
              // holds columns 8 lk .. 8 lk + 7 of the 32 that two sub-tiles make
        static_assert(EPI != EPI_SWIGLU || D::NI % 4 == 0, "SwiGLU epilogue pairs 32-column blocks");
        const int half_n = N / 2;
        bf16_t* out = g.out_bf16 + col0 / 2 + 8 * lk;
#pragma unroll
        for (int mi = 0; mi < D::MI; ++mi) {
            const int m = row0 + mi * 16;
            if (m >= M) continue;
            u32x4_a2* dst = reinterpret_cast<u32x4_a2*>(out + (size_t)m * half_n);
#pragma unroll
            for (int j = 0; j < D::NI / 4; ++j) {
                if (!inside(4 * j)) continue;
                float y[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float gt = acc[mi][4 * j + e / 4][e % 4], up = acc[mi][4 * j + 2 + e / 4][e % 4];
                    y[e] = gt / (1.f + __expf(-gt)) * up;
                }
                u32x4 w;
#pragma unroll
                for (int e = 0; e < 4; ++e) w[e] = pack_bf16x2(y[2 * e], y[2 * e + 1]);
                dst[j * 4] = w;
            }
        }
    }
}

// The matrix instructions are inline assembly: the builtin has separate accumulator operands in and out, and the register
// allocator fills the loop with moves between them.  The compiler therefore does not know the wait states between them and
// what else touches their accumulators: 2 after a vector instruction wrote one, 11 before one reads it.  Every accumulator
// passes through a statement behind the wait, so that no access can be placed before it.
template <typename D>
__device__ __forceinline__ void acc_fence(f32x4 (&acc)[D::MI][D::NI]) {
    asm volatile("s_nop 15\n\ts_nop 7" ::: "memory");
#pragma unroll
    for (int mi = 0; mi < D::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < D::NI; ++ni) {
            if (D::in_vgpr(mi, ni)) asm volatile("" : "+v"(acc[mi][ni]));
            else asm volatile("" : "+a"(acc[mi][ni]));
        }
}

template <int V>
constexpr std::integral_constant<int, V> I{};

// all but the last N loads of this wave have landed and its LDS reads are done; so are the other waves'
template <int N>
__device__ __forceinline__ void dma_barrier() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// One tile of the rows_in live rows: workgroup `bid` of tiles_m * tiles_n * g.split.  late_live: NULL, or where the number
// of live rows is found if it does not decide which tile this is (a single row tile): it is then read behind the first
// weight loads.
template <int BM, int BN, int WM, int WN, int EPI, bool STREAM>
__device__ __forceinline__ void dma_tile(const GemmArgs& g, unsigned char* smem, const int rows_in, const int tiles_m,
                                         const int tiles_n, const int bid, const int* late_live) {
    using D = DmaTraits<BM, BN, WM, WN>;
    constexpr int MH = D::MI / 2, NH = D::NI / 2, NS = D::NS;
    constexpr bool PAIRED = EPI == EPI_SWIGLU;
    const int K = g.K;
    const TileCoord tc = map_block(bid, tiles_m, tiles_n, g.split);
    const int m0 = tc.tm * BM, n0 = tc.tn * BN;
    const int kbeg = tc.ks * g.kps;
    const int kend = (kbeg + g.kps < K) ? (kbeg + g.kps) : K;
    const int KT = (kend - kbeg) / BK;
    const int tid = threadIdx.x;
    if (g.row_live != nullptr) {  // a row tile made of padding only has nothing to compute (and nothing reads its output)
        bool any = false;
        for (int r = tid; r < BM; r += 256) any |= (m0 + r < rows_in) && g.row_live[m0 + r] >= 0;
        int* flag = reinterpret_cast<int*>(smem);
        const bool wave_any = __builtin_amdgcn_ballot_w64(any) != 0;
        if ((tid & 63) == 0) flag[tid >> 6] = wave_any;
        __syncthreads();
        int live = 0;
#pragma unroll
        for (int w = 0; w < 4; ++w) live |= flag[w];
        if (!live) return;
        __syncthreads();
    }
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave / WN, wn = wave % WN;
    const int lrow = lane & 15, lk = lane >> 4;

    const unsigned row_bytes = (unsigned)K * 2u;
    auto rsrc = [&](const bf16_t* base, unsigned bytes) {
        const unsigned long long p = reinterpret_cast<unsigned long long>(base);
        return i32x4{__builtin_amdgcn_readfirstlane((int)(unsigned)p), __builtin_amdgcn_readfirstlane((int)(p >> 32)),
                     __builtin_amdgcn_readfirstlane((int)bytes), 0x00020000};
    };
    i32x4 ra, rb = rsrc(g.W + (size_t)n0 * K, (unsigned)(D::RAGGED && g.cols - n0 < BN ? g.cols - n0 : BN) * row_bytes);
    int a_bytes, b_bytes = rb[2];
    // Offsets of a lane's chunks: half slab row q -> tile row (q / (WT/2)) * WT + half * WT/2 + q % (WT/2).  Rows of A past the
    // last one lie behind the descriptor's end and padding rows are sent there: no request is made for them (a unit keeps a
    // bounded number in flight, and A takes a third of it on 128 x 256).  So each row of A has an offset of its own.  On 320 x 256 there are no registers for as
    // many of B: the rows that share a key share one there, and the scalar offset moves it (a 256-row graph of the 7B layer is
    // 2.5 % slower where all tiles do that).
    constexpr bool SHARE = BM > 256;
    constexpr int KEYS = SHARE ? (PAIRED ? 4 : 2) : D::LB;
    unsigned va[2][D::LA], vb[SHARE ? 1 : 2][KEYS];
    {
        const int qa = wave * D::QA, qb = wave * D::QB;
        const int ta = qa / (D::WTM / 2) * D::WTM + qa % (D::WTM / 2), tb = qb / (D::WTN / 2) * D::WTN + qb % (D::WTN / 2);
        const int r = lane >> 3, c = lane & 7;
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < D::LA; ++i) {
                const int row = ta + h * D::WTM / 2 + 8 * i + r;
                va[h][i] = (unsigned)row * row_bytes + (c ^ dma_key<false>(qa + 8 * i + r)) * 16 + (unsigned)kbeg * 2u;
                if (g.row_live != nullptr && m0 + row < rows_in && g.row_live[m0 + row] < 0) va[h][i] = 0xf0000000u;
            }
#pragma unroll
        for (int h = 0; h < (SHARE ? 1 : 2); ++h)
#pragma unroll
            for (int i = 0; i < KEYS; ++i)
                vb[h][i] = (unsigned)(tb + r + (SHARE ? 0 : h * D::WTN / 2 + 8 * i)) * row_bytes + (c ^ dma_key<PAIRED>(qb + 8 * i + r)) * 16 + (unsigned)kbeg * 2u;
    }
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const unsigned lds_a = lds0 + wave * D::QA * 128, lds_b = lds0 + D::HA * 128 + wave * D::QB * 128;
    // load i of half slab (kt, A rows ha, B rows hb) into the slot at byte `slot`
    auto dma = [&](int i, int ha, int hb, unsigned slot, int koff) {
        if (i < D::LA) {
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                         ::"s"(lds_a + slot + i * 1024), "v"(va[ha][i]), "s"(ra), "s"(koff));
            return;
        }
        const int j = i - D::LA, off = SHARE ? koff + (hb * (D::WTN / 2) + 8 * j) * (int)row_bytes : koff;
        const unsigned lane_off = vb[SHARE ? 0 : hb][j % KEYS];
        if (STREAM && (D::QB % 8 == 0 || j < D::LB - 1))
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen nt lds"
                         ::"s"(lds_b + slot + j * 1024), "v"(lane_off), "s"(rb), "s"(off));
        else if (D::QB % 8 == 0 || j < D::LB - 1)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                         ::"s"(lds_b + slot + j * 1024), "v"(lane_off), "s"(rb), "s"(off));
        else   // four rows: the first 32 lanes
            asm volatile("s_mov_b32 m0, %0\n\ts_mov_b32 exec_hi, 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds\n\ts_mov_b32 exec_hi, -1"
                         ::"s"(lds_b + slot + j * 1024), "v"(lane_off), "s"(rb), "s"(off));
    };

    f32x4 acc[D::MI][D::NI];
#pragma unroll
    for (int mi = 0; mi < D::MI; ++mi)
#pragma unroll
        for (int ni = 0; ni < D::NI; ++ni) acc[mi][ni] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 fa[2][D::MI], fb[2][D::NI];   // [k-step of 32]
    const u32x4* L = reinterpret_cast<const u32x4*>(smem);
    const int key = (lrow >> 1) & 7;
    const int src_a = (wm * (D::WTM / 2) + lrow) * CHUNKS;
    const int src_b = (D::HA + wn * (D::WTN / 2) + (PAIRED ? 8 * (lrow >> 2) + (lrow & 3) : lrow)) * CHUNKS;
    auto read_a = [&](int h, int i, unsigned slot) {   // i < 2 MH: k-step i / MH
        const int kk = i / MH, mi = i % MH;
        fa[kk][h * MH + mi] = __builtin_bit_cast(bf16x8, L[slot / 16 + src_a + mi * 16 * CHUNKS + ((lk + kk * 4) ^ key)]);
    };
    auto read_b = [&](int h, int i, unsigned slot) {
        const int kk = i / NH, ni = i % NH, row = PAIRED ? ni / 2 * 32 + ni % 2 * 4 : ni * 16;
        fb[kk][h * NH + ni] = __builtin_bit_cast(bf16x8, L[slot / 16 + src_b + row * CHUNKS + ((lk + kk * 4) ^ key)]);
    };

    // Products of a slab: four quadrants of the wave's tile, each with one new half of A or B:
    //   even slabs   A0B0 | read B1,  A0B1 | read A1,  A1B1 | read the next slab's A0,  A1B0 | read its B1
    //   odd slabs    A0B1 | read B0,  A0B0 | read A1,  A1B0 | read the next slab's A0,  A1B1 | read its B0
    // Half slab p is what quadrants 2p - 2 and 2p - 1 read: A half p % 2 and B half (p ^ (p >> 1)) & 1 of slab p / 2.  While
    // half slab p is multiplied, p + 1 is read and p + NS is loaded into the place of p.
    int M = rows_in;
    if (STREAM) {
#pragma unroll
        for (int i = D::LA; i < D::LOADS; ++i) dma(i, 0, 0, 0, 0);
        if (late_live != nullptr) {
            // A scalar load: behind the requests above the compiler makes a vector load of a plain read, which returns in order
            // and so waited for the first weights before anything else was requested (14B replay of 8 rows 134.9 -> 133.1 us, four
            // 32B layers of 128 rows 882 -> 876).
            int live;
            asm volatile("s_load_dword %0, %1, 0x0\n\ts_waitcnt lgkmcnt(0)" : "=&s"(live) : "s"(late_live));
            M = live < M ? live : M;
            if (M <= 0) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // as at the end
                return;
            }
        }
    }
    ra = rsrc(g.A + (size_t)m0 * K, (unsigned)(M - m0 < BM ? M - m0 : BM) * row_bytes);
    a_bytes = ra[2];
    // Slabs past the last one are loaded from descriptors of no bytes, which takes no request (with the last slab again in
    // their place q/k/v of 128 rows took 22.5 us instead of 21.0, down 58 instead of 54).  Not where power bounds: there the
    // loads of the last slab again cost nothing, and a 4096-row graph took 0.7 % longer without them.
    auto until = [&](int k) {
        if (STREAM) {
            ra[2] = k < KT ? a_bytes : 0;
            rb[2] = k < KT ? b_bytes : 0;
        }
        return (k < KT ? k : KT - 1) * (BK * 2);
    };
#pragma unroll
    for (int i = 0; i < (STREAM ? D::LA : D::LOADS); ++i) dma(i, 0, 0, 0, 0);
#pragma unroll
    for (int p = 1; p < NS; ++p) {
        const int koff = until(p / 2);
#pragma unroll
        for (int i = 0; i < D::LOADS; ++i) dma(i, p & 1, (p ^ (p >> 1)) & 1, p * D::SLOT, koff);
    }
    dma_barrier<(NS - 1) * D::LOADS>();
#pragma unroll
    for (int i = 0; i < 2 * MH; ++i) read_a(0, i, 0);
#pragma unroll
    for (int i = 0; i < 2 * NH; ++i) read_b(0, i, 0);
    acc_fence<D>(acc);
    dma_barrier<(NS - 2) * D::LOADS>();

    unsigned rd = D::SLOT, wr = 0;   // places of half slabs p + 1 and p
    // One quadrant: rows half ma times columns half nb, both k-steps.  Spread over the first three quarters of its matrix
    // instructions, so that the barrier finds the reads done: the fragments of half rh of A or B, and loads [l0, l1) of half
    // slab p + NS (halves ha, hb).
    auto quadrant = [&](auto ma, auto nb, auto rd_a, auto rh, auto l0, auto l1, auto ha, auto hb, int koff) {
        constexpr int NM = 2 * MH * NH, SPAN = NM * 3 / 4;
        constexpr int NR = rd_a() ? 2 * MH : 2 * NH, NL = l1() - l0(), OPS = NR + NL;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int kk = i / (MH * NH), nr = i % (MH * NH) / MH;
            const int mi = ma() * MH + (nr & 1 ? MH - 1 - i % MH : i % MH), ni = nb() * NH + nr;
            if (D::in_vgpr(mi, ni))
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(acc[mi][ni]) : "v"(fb[kk][ni]), "v"(fa[kk][mi]));
            else
                asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(acc[mi][ni]) : "v"(fb[kk][ni]), "v"(fa[kk][mi]));
            const int j0 = i < SPAN ? i * OPS / SPAN : OPS, j1 = i + 1 < SPAN ? (i + 1) * OPS / SPAN : OPS;
#pragma unroll
            for (int j = j0; j < j1; ++j) {
                const int nl = j * NL / OPS;   // loads among the operations before j
                if ((j + 1) * NL / OPS > nl) dma(l0() + nl, ha(), hb(), wr, koff);
                else if (rd_a()) read_a(rh(), j - nl, rd);
                else read_b(rh(), j - nl, rd);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto next = [&](unsigned s) { return s + D::SLOT == NS * D::SLOT ? 0u : s + D::SLOT; };
    auto half_end = [&]() {
        dma_barrier<(NS - 2) * D::LOADS>();
        __builtin_amdgcn_sched_barrier(0);
        wr = rd;
        rd = next(rd);
        if (SHARE) asm volatile("" : "+s"(rd), "+s"(wr));   // one address per operand and k-step, not one for every place of the ring
    };
    auto slab = [&](auto parity, int kt) {
        constexpr int B = decltype(parity)::value;   // the columns half this slab begins with
        constexpr int P0 = 2 * B, P1 = 2 * B + 1;    // p modulo 4
        constexpr int N0 = (P0 + NS) & 3, N1 = (P1 + NS) & 3, H0 = (N0 ^ (N0 >> 1)) & 1, H1 = (N1 ^ (N1 >> 1)) & 1;
        constexpr int LH = D::LOADS / 2;
        const int o0 = until(kt + NS / 2);           // half slab p + NS lies in slab (p + NS) / 2
        quadrant(I<0>, I<B>, I<0>, I<B ^ 1>, I<0>, I<LH>, I<(N0 & 1)>, I<H0>, o0);
        quadrant(I<0>, I<B ^ 1>, I<1>, I<1>, I<LH>, I<D::LOADS>, I<(N0 & 1)>, I<H0>, o0);
        half_end();
        const int o1 = until(kt + (1 + NS) / 2);
        quadrant(I<1>, I<B ^ 1>, I<1>, I<0>, I<0>, I<LH>, I<(N1 & 1)>, I<H1>, o1);
        quadrant(I<1>, I<B>, I<0>, I<B ^ 1>, I<LH>, I<D::LOADS>, I<(N1 & 1)>, I<H1>, o1);
        half_end();
    };
    for (int kt = 0;;) {
        slab(I<0>, kt);
        if (++kt >= KT) break;
        slab(I<1>, kt);
        if (++kt >= KT) break;
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // no load may land after this workgroup's LDS is another's
    acc_fence<D>(acc);
    if (D::RAGGED && __builtin_expect(n0 + BN > g.cols, 0)) store_dma_tile<D, EPI, true>(acc, g, M, tc.ks, m0, n0, wm, wn, lrow, lk);
    else store_dma_tile<D, EPI, false>(acc, g, M, tc.ks, m0, n0, wm, wn, lrow, lk);
}

// Rows past *n_live are padding: the tiles of the rows before them are dealt out as if there were no others.  (Tiles of all
// M rows, the dead ones returning at once, leave whole XCDs idle, since each takes a contiguous range: gate/up of a
// 4096-row graph with 2776 live rows 1880 us, this way 1390, both with slabs through registers.)
__device__ __forceinline__ int live_rows(const GemmArgs& g) {
    if (g.n_live == nullptr) return g.M;
    const int live = *g.n_live;
    return live < g.M ? live : g.M;
}

template <int BM, int BN, int WM, int WN, int EPI, int WS>
__global__ __launch_bounds__(WM* WN * 64, (Traits<BM, BN, WM, WN>::WAVES_PER_SIMD)) void far_kernel(const GemmArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int M = live_rows(g), tiles_m = (M + BM - 1) / BM;
    if (M <= 0 || (int)blockIdx.x >= tiles_m * g.tiles_n * g.split) return;
    far_tile<BM, BN, WM, WN, EPI, WS>(g, smem, M, tiles_m, g.tiles_n, blockIdx.x);
}

// STREAM: nobody else reads this tile's weights (a single row tile), they bypass the caches.
template <int BM, int BN, int WM, int WN, int EPI, bool STREAM>
__global__ __launch_bounds__(256, (DmaTraits<BM, BN, WM, WN>::TWO ? 2 : 1)) void dma_kernel(const GemmArgs g) {
    extern __shared__ __align__(16) unsigned char smem[];
    if (STREAM) {   // the live rows do not decide which tile this is
        dma_tile<BM, BN, WM, WN, EPI, true>(g, smem, g.M, 1, g.tiles_n, blockIdx.x, g.n_live);
        return;
    }
    const int M = live_rows(g), tiles_m = (M + BM - 1) / BM;
    if (M <= 0 || (int)blockIdx.x >= tiles_m * g.tiles_n * g.split) return;
    dma_tile<BM, BN, WM, WN, EPI, false>(g, smem, M, tiles_m, g.tiles_n, blockIdx.x, nullptr);
}

// Plans that the fit of kTiles' cost columns has not seen have to lead on paper by more than it errs on them.  Measured against
// the plan without them, products of the 7B, 14B and 32B projections and of 19 other weights (1536 x 8960 to 57344 x 8192), 129
// to 11104 rows, then of 20 weights and 60 row counts that the lines were not drawn with:
//   a last column tile past n: 1.01 to 1.22 times as fast (61 products); 1.02 to 1.45 of the others (90), one 0.98;
//   192 rows where they need more row tiles than 256: 0.995 to 1.23 from a lead of 6 % on (52), 0.93 to 1.10 below (30: 2560
//   columns, K = 9728, 1138 rows 61.7 -> 66.7 us); 1.01 to 1.36 of the others (45), one 0.97;
//   whole rounds and smaller tiles behind them: 0.993 to 1.29 from 4 % on, 0.95 to 1.03 below; 0.99 to 1.30 of the others (276),
//   three of them, 2304 and 3072 columns of more than 7000 rows, 0.977 to 0.986.
constexpr double kRaggedMargin = 1.085, kMore192Margin = 1.06, kMixMargin = 1.04;

// A captured graph is launched for all its rows, and the tile that fills the chip for them (down projection, 4096 rows:
// 512 tiles of 256 x 160 in two rounds) is not the one for the rows a batch has (2776: 352 tiles in two rounds where 253
// of 256 x 224 take one: 997 against 700 us with slabs through registers on 256 x 256; 612 on 256 x 256 and 581 on 256 x 224
// now).  The tiles of one workgroup a unit are therefore one kernel, which takes the one that the cost model gives the live
// rows; every workgroup comes to the same choice.  The last column tile may reach past N, so that every width serves every N.
// q/k/v of 2776 rows on 320 x 256 (252 tiles, one round) 152 us, on 256 x 224 (352) 198; gate/up 1141 on 320 x 256 and 1178 on
// 256 x 256; 7B o on 256 x 160 (253 tiles) 81, on 256 x 224 (176) 93.
constexpr int kLiveTiles = 7;
constexpr int kLiveRows[kLiveTiles] = {256, 256, 256, 320, 192, 256, 256}, kLiveCols[kLiveTiles] = {256, 128, 192, 256, 256, 224, 160};
constexpr int live_tiles(int epi) { return epi == EPI_SWIGLU ? 5 : 7; }   // no gate / up pairs in a wave of the last two
struct LiveCost {
    float fill[kLiveTiles], slabs[kLiveTiles], part[kLiveTiles];   // as TileDef, slabs = time of all K slabs on a full chip
};
template <int EPI>
__global__ __launch_bounds__(256, 1) void gemm_live_kernel(const GemmArgs g, const LiveCost c) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int M = live_rows(g);
    if (M <= 0) return;
    int pick = 0;
    float best = 0.f;
#pragma unroll
    for (int i = 0; i < live_tiles(EPI); ++i) {
        const int tiles_m = (M + kLiveRows[i] - 1) / kLiveRows[i], tiles = tiles_m * ((g.N + kLiveCols[i] - 1) / kLiveCols[i]);
        const float spare = tiles < 256 ? 1.f - tiles / 256.f : 0.f;
        float us = (float)((tiles + 255) / 256) * (c.fill[i] + c.slabs[i] * (1.f - c.part[i] * spare));
        if (g.N % kLiveCols[i] != 0) us *= (float)kRaggedMargin;   // as in laps_gemm_plan
        else if (kLiveRows[i] == 192 && tiles_m != (M + 255) / 256) us *= (float)kMore192Margin;
        if (i == 0 || us < best) best = us, pick = i;
    }
    int rows = kLiveRows[0], cols = kLiveCols[0];
#pragma unroll
    for (int i = 1; i < live_tiles(EPI); ++i)
        if (pick == i) rows = kLiveRows[i], cols = kLiveCols[i];
    const int tiles_m = (M + rows - 1) / rows, tiles_n = (g.N + cols - 1) / cols;
    if ((int)blockIdx.x >= tiles_m * tiles_n) return;
    if constexpr (EPI != EPI_SWIGLU) {
        if (pick == 5) return dma_tile<256, 224, 4, 1, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
        if (pick == 6) return dma_tile<256, 160, 4, 1, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
    }
    if (pick == 0) dma_tile<256, 256, 2, 2, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
    else if (pick == 1) dma_tile<256, 128, 2, 2, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
    else if (pick == 2) dma_tile<256, 192, 4, 1, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
    else if (pick == 3) dma_tile<320, 256, 2, 2, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
    else dma_tile<192, 256, 2, 2, EPI, false>(g, smem, M, tiles_m, tiles_n, blockIdx.x, nullptr);
}

// Whole rounds of big tiles over the compute units, and the columns that they leave in smaller tiles behind them: a last round
// of a few big tiles takes as long as a full one.  `big` workgroups of 256 x 256 (320 x 256 if tall) on g, the others on h, the
// columns behind g's; small: 0 = 128 x 128, 1 = 192 x 128, 2 = 256 x 128, one workgroup a unit beside the big tiles' registers.
// What a few tiles in the last round cost, SwiGLU, K = 5120: 1847 rows of 55296 columns, 1296 tiles of 320 x 256 in 5.06 rounds,
// 772 us; 1278 of them and 90 of 128 x 128 724.  1024 rows of 37888 columns, K = 3584, 592 tiles of 256 x 256 239 us; 512 and 240
// of 192 x 128 202.  The sums are the same bits: every tile walks K alike.
constexpr int kMixRows[3] = {128, 192, 256};
template <int EPI>
__global__ __launch_bounds__(256, 1) void gemm_mix_kernel(const GemmArgs g, const GemmArgs h, const int big, const int tall, const int small) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int M = live_rows(g), bid = blockIdx.x;
    if (M <= 0) return;
    if (bid < big) {
        const int rows = tall ? 320 : 256, tiles_m = (M + rows - 1) / rows;
        if (bid >= tiles_m * g.tiles_n) return;
        if (tall) dma_tile<320, 256, 2, 2, EPI, false>(g, smem, M, tiles_m, g.tiles_n, bid, nullptr);
        else dma_tile<256, 256, 2, 2, EPI, false>(g, smem, M, tiles_m, g.tiles_n, bid, nullptr);
        return;
    }
    const int rows = small == 0 ? kMixRows[0] : small == 1 ? kMixRows[1] : kMixRows[2], tiles_m = (M + rows - 1) / rows;
    if (bid - big >= tiles_m * h.tiles_n) return;
    if (small == 0) dma_tile<128, 128, 2, 2, EPI, false>(h, smem, M, tiles_m, h.tiles_n, bid - big, nullptr);
    else if (small == 1) dma_tile<192, 128, 2, 2, EPI, false>(h, smem, M, tiles_m, h.tiles_n, bid - big, nullptr);
    else dma_tile<256, 128, 2, 2, EPI, false>(h, smem, M, tiles_m, h.tiles_n, bid - big, nullptr);
}

int launch_gemm(void (*kern)(const GemmArgs), bool* attr_set, int threads, int lds, const GemmArgs& a, hipStream_t s) {
    if (!*attr_set) {   // per kernel; idempotent, so a race only repeats the call
        LAPS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        *attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(a.tiles_m * a.tiles_n * a.split), dim3(threads), lds, s, a);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

template <int BM, int BN, int WM, int WN, int EPI, int WS>
int launch_far(const GemmArgs& a, hipStream_t s) {
    static bool attr_set = false;
    return launch_gemm(far_kernel<BM, BN, WM, WN, EPI, WS>, &attr_set, Traits<BM, BN, WM, WN>::NT, Traits<BM, BN, WM, WN>::LDS_BYTES, a, s);
}

template <int BM, int BN, int WM, int WN, int EPI, bool STREAM>
int launch_dma(const GemmArgs& a, hipStream_t s) {
    static bool attr_set = false;
    return launch_gemm(dma_kernel<BM, BN, WM, WN, EPI, STREAM>, &attr_set, 256, DmaTraits<BM, BN, WM, WN>::LDS, a, s);
}

template <int BM, int BN, int WM, int WN, bool STREAM>
int launch_dma_epi(int epi, const GemmArgs& a, hipStream_t s) {
    using D = DmaTraits<BM, BN, WM, WN>;
    if (epi == EPI_PARTIAL) return launch_dma<BM, BN, WM, WN, EPI_PARTIAL, STREAM>(a, s);
    if (epi == EPI_RESID) return launch_dma<BM, BN, WM, WN, EPI_RESID, STREAM>(a, s);
    if constexpr (D::NI % 4 == 0) return launch_dma<BM, BN, WM, WN, EPI_SWIGLU, STREAM>(a, s);
    laps_set_error("gemm: no SwiGLU on a tile of %d columns", BN);
    return LAPS_EINVAL;
}

struct TileDef {
    int bm, bn;
    int ws;            // slabs that a K slice holds a multiple of where K allows it (far_tile's loop needs it on 192 x 256; the
                       // others walk any number and share the rule, which laps_gemm_plan_info reports)
    double fill, slab, part;   // cost model of launches above 128 rows, see laps_gemm_plan
};
// index = GemmPlan::cfg.  The cost columns are a fit over 4800 launches (all tiles and K splits on the 7B, 14B and 32B
// projections at 24 row counts from 129 to 8192, weights cold; rms error 7 %): microseconds a workgroup takes besides its
// slabs, microseconds per 64-wide K slab on a full chip, and the share of the latter that goes away on an empty one.  Fitted
// with slabs through registers, as are the choices; against the best plan of each of 100 products (ten projections at ten row
// counts, all tiles of up to 256 rows and all splits, slabs straight into LDS) they cost 1.1 % in the mean, over 4 % in ten of
// them and 23 % at worst (a 7168 x 5120 product of its own, 1000 rows: 75 us in one slice of 256 x 128, 61 in two of 256 x 224,
// which the layer takes).
constexpr TileDef kTiles[] = {
    {128, 128, 2, 1.11, 0.521, 0.06},  // 0: 4 waves of 64x64 (32x64 up to 64 rows), two workgroups per compute unit
    {128, 64, 2, 1.20, 0.350, 0.00},   // 1: 4 waves of 64x32, for n % 128 != 0
    {256, 256, 2, 5.25, 1.430, 0.25},  // 2: 4 waves of 128x128
    {256, 224, 2, 5.19, 1.234, 0.24},  // 3: 4 waves of 64x224 (N = 7168 -> 32 column tiles)
    {256, 160, 2, 4.38, 0.985, 0.24},  // 4: 4 waves of 64x160 (N = 5120 -> 32 column tiles)
    {128, 256, 2, 2.44, 0.904, 0.21},  // 5: 4 waves of 128x64 (64x64 up to 64 rows): the streaming tile, A slab shared by 256 columns
    {192, 256, 2, 5.75, 1.160, 0.20},  // 6: 4 waves of 96x128
    {192, 128, 1, 1.81, 0.716, 0.09},  // 7: 4 waves of 96x64, two workgroups per compute unit
    {256, 128, 2, 3.01, 0.863, 0.25},  // 8: 4 waves of 128x64
    {256, 192, 2, 2.93, 1.199, 0.31},  // 9: 4 waves of 64x192 (N = 55296, 27648, 4608)
    {320, 256, 1, 6.83, 1.597, 0.11},  // 10: 4 waves of 160x128, inside layers; fitted to 400 launches against the others
};
constexpr int kNumTiles = sizeof(kTiles) / sizeof(kTiles[0]);

// The tiles behind whole rounds of big ones, alone on their compute unit: cost as above, without `part`.  Fitted to 467 products
// (the first ones above kRaggedMargin), which they meet within 4 % (rms).  The first constants, from 84 products, had 128 x 128 at
// half its time: 14B down of 3396 rows, 256 x 160 in 1.75 rounds, 402 -> 414 us.
struct MixDef {
    int cfg;
    double fill, slab;
};
constexpr MixDef kMix[3] = {{0, 8.0, 0.60}, {7, 6.0, 0.80}, {8, 2.0, 1.00}};   // in the order of kMixRows

template <int EPI>
int launch_live(const GemmArgs& a, hipStream_t s) {
    constexpr int cfg[kLiveTiles] = {2, 8, 9, 10, 6, 3, 4};   // in the order of kLiveRows, kLiveCols
    constexpr int lds_of[kLiveTiles] = {DmaTraits<256, 256, 2, 2>::LDS, DmaTraits<256, 128, 2, 2>::LDS, DmaTraits<256, 192, 4, 1>::LDS,
                                        DmaTraits<320, 256, 2, 2>::LDS, DmaTraits<192, 256, 2, 2>::LDS, DmaTraits<256, 224, 4, 1>::LDS,
                                        DmaTraits<256, 160, 4, 1>::LDS};
    int lds = 0, most = 0;   // the most tiles of any choice
    LiveCost c;
    for (int i = 0; i < live_tiles(EPI); ++i) {
        lds = lds_of[i] > lds ? lds_of[i] : lds;
        const int tiles = (a.M + kLiveRows[i] - 1) / kLiveRows[i] * ((a.N + kLiveCols[i] - 1) / kLiveCols[i]);
        most = tiles > most ? tiles : most;
    }
    for (int i = 0; i < kLiveTiles; ++i) {
        c.fill[i] = (float)kTiles[cfg[i]].fill;
        c.slabs[i] = (float)(kTiles[cfg[i]].slab * (a.K / BK));
        c.part[i] = (float)kTiles[cfg[i]].part;
    }
    auto kern = gemm_live_kernel<EPI>;
    static bool attr_set = false;  // as in launch_gemm
    if (!attr_set) {
        LAPS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds));
        attr_set = true;
    }
    hipLaunchKernelGGL(kern, dim3(most), dim3(256), lds, s, a, c);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

// Column tiles of 256 that whole rounds of the big tiles take.
int mix_columns(int tiles_m, int n) { return (int)((long)tiles_m * (n / 256) / 256 * 256 / tiles_m); }

template <int EPI>
int launch_mix(const GemmArgs& a, bool tall, int small, hipStream_t s) {
    const int lds_big = tall ? DmaTraits<320, 256, 2, 2>::LDS : DmaTraits<256, 256, 2, 2>::LDS;
    constexpr int lds_small[3] = {DmaTraits<128, 128, 2, 2>::LDS, DmaTraits<192, 128, 2, 2>::LDS, DmaTraits<256, 128, 2, 2>::LDS};
    constexpr int lds_most = DmaTraits<256, 256, 2, 2>::LDS > DmaTraits<320, 256, 2, 2>::LDS ? DmaTraits<256, 256, 2, 2>::LDS : DmaTraits<320, 256, 2, 2>::LDS;
    static_assert(lds_small[2] <= lds_most && lds_small[1] <= lds_most, "the attribute below covers every tile");
    GemmArgs g = a, h = a;
    g.tiles_n = mix_columns(a.tiles_m, a.N);
    g.cols = g.tiles_n * 256;
    h.cols = a.N - g.cols;
    h.tiles_n = (h.cols + 127) / 128;
    h.tiles_m = (a.M + kMixRows[small] - 1) / kMixRows[small];
    h.W = a.W + (size_t)g.cols * a.K;
    if (a.out_f32) h.out_f32 = a.out_f32 + g.cols;
    if (a.resid) h.resid = a.resid + g.cols;
    if (a.out_bf16) h.out_bf16 = a.out_bf16 + g.cols / 2;
    auto kern = gemm_mix_kernel<EPI>;
    static bool attr_set = false;  // as in launch_gemm
    if (!attr_set) {
        LAPS_HIP(hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds_most));
        attr_set = true;
    }
    const int big = g.tiles_m * g.tiles_n;
    hipLaunchKernelGGL(kern, dim3(big + h.tiles_m * h.tiles_n), dim3(256), lds_big > lds_small[small] ? lds_big : lds_small[small], s, g, h, big,
                       (int)tall, small);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

}  // namespace

void laps_gemm_tile_dims(int cfg, int* bm, int* bn) {
    *bm = (cfg >= 0 && cfg < kNumTiles) ? kTiles[cfg].bm : 0;
    *bn = (cfg >= 0 && cfg < kNumTiles) ? kTiles[cfg].bn : 0;
}

// Picks tile shape and K split.
GemmPlan laps_gemm_plan(int m, int n, int k, int force_split, int want_epi, size_t partial_cap, bool row_kernel, bool layer) {
    GemmPlan p;
    const int ksteps = k / BK;
    const bool far = k >= kMaxBufferK;   // rows that only the pointer-addressed tiles (1, 6, 7) reach
    if (far && want_epi == EPI_SWIGLU && n % 128 != 0) want_epi = EPI_PARTIAL;
    auto finish = [&](int cfg, int split) {
        if (split > ksteps) split = ksteps;
        if (split < 1) split = 1;
        int per = (ksteps + split - 1) / split;
        p.ws = 1;
        if (kTiles[cfg].ws == 2 && ksteps % 2 == 0 && !(far && cfg == 1)) {
            per = (per + 1) / 2 * 2;
            p.ws = 2;
        }
        p.cfg = cfg;
        p.rest = 0;
        p.k_per_split = per * BK;
        p.split = (ksteps + per - 1) / per;
        p.epi = (p.split == 1) ? want_epi : EPI_PARTIAL;
        return p;
    };
    if (m <= 128 && !far) {
        // Bandwidth-bound.  A CU keeps a bounded number of requests in flight, and the A slab that every
        // workgroup re-reads per K step (L2 hits) takes its share of them from the weight stream: a
        // 256-column tile halves the A share of a 128-column one, which decides the wide projections
        // (32B gate/up of 128 rows: 104 against 126 us).  A narrow
        // projection (q/k/v, o: 20-28 tiles of 256 columns) never gets near that limit; it pays for the
        // K split that has to fill the chip - every slice writes m*n fp32 partial sums that a reduce
        // kernel reads back - and for the short pipeline of each slice.  128-column tiles need half the
        // split; they win where the 256-column slices would be shorter than 24 K slabs (cold
        // weights, m = 128: q/k/v 22.2 -> 21.3 us, o with the row kernel 30.2 -> 26.2, 7B down 43.0 -> 39.9;
        // the 32B down projection, 36 slabs per slice, stays on 256 columns: 61.2 against 65.8).  At most 256
        // workgroups either way: a streaming kernel with 257 leaves one CU with twice the work.
        auto auto_split = [&](int c) {
            // Slices of 16 slabs or more: below, the pipeline is all prologue.  8 where a row kernel reads the sums anyhow (q/k/v
            // in the 7B layer at 8 / 128 rows: 4 slices of 14 slabs 8.7 / 15.1 us, 7 of 8 7.6 / 12.6).  Raw sums of a product of
            // its own are its result if K is one slice, and cost a launch and a workspace if not (3584 columns, K = 768, 128
            // rows: one slice 11.1, two 13.1); where 16 slabs split K already, up to 4 slices of 8 pay, and more until they fill
            // half the chip (48 rows: 512 x 2560 3 slices 12.4, 5 8.9; 2048 x 3584 4 slices 12.0, 7 10.8; 7168 x 1920, 64 rows,
            // 2 slices 17.1, 4 14.2; but 4608 x 3584 4 slices 14.2, 7 16.1).
            const int tiles = n / kTiles[c].bn, fine = (ksteps + 4) / 8;
            int sp = 256 / tiles, cap = (ksteps + 8) / 16;
            const bool read_anyhow = want_epi != EPI_SWIGLU && row_kernel;
            // Above 64 rows two tiles of 64 in half the slices (laps_gemm_launch) where those are 3 or more, and the shorter the fewer
            // rows of A one tile would take in: up to 12 + m / 12 slabs.  With the row kernel, 32 products of 1536 to 7168 columns and
            // K = 1536 to 8192 at 7 row counts from 66 to 128: no pair that this takes is behind the one tile (7B q/k/v at 80 / 96 / 128
            // rows in 7 slices 17.5 / 18.9 / 21.4, in 3 17.0 / 17.9 / 19.1; 3584 x 5120, 20 slabs, at 66 / 96 / 128 rows in 8 16.6 / 19.4 /
            // 22.3, in 4 17.3 / 18.8 / 20.4), and all of them are within 1 % of the best in the mean (one tile 3.6).
            const int halves = std::min(128 / tiles, fine);
            if (c == 0 && m > 64 && read_anyhow && halves >= 3 && 12 * ksteps <= (144 + m) * halves) return halves;
            // Residual products up to 64 rows split at 16 slabs already: finer slices are read by the same row kernel, and pay where the
            // longest is shorter by a third (same products, 1 to 64 rows: 0.99 to 1.28 times as fast, 2048 x 2048 at 8 / 64 rows 11.0 /
            // 13.1 us in 2, 8.7 / 10.7 in 4; 16 slabs in 12 lose, 5120 x 4096 13.4 / 17.4 in 4 and 14.1 / 17.9 in 6).  Above 64 rows they
            // lose (4096 x 6144 at 72 / 128 rows 18.9 / 23.6 in 6, 19.5 / 25.1 in 8) or are even (32B o, 128 rows, alone 24.8 in 5 and
            // 25.1 in 6, in a graph of four layers 1 us the other way round).
            const auto longest = [&](int split) {
                const int per = (ksteps + split - 1) / split;
                return ksteps % 2 == 0 ? (per + 1) / 2 * 2 : per;
            };
            const bool finer = want_epi == EPI_PARTIAL || (cap > 1 && m <= 64 && 3 * longest(std::min(sp, fine)) <= 2 * longest(std::min(sp, cap)));
            if (c == 5 || (read_anyhow && finer)) cap = fine;
            else if (want_epi == EPI_PARTIAL && cap > 1) cap = std::max(cap, std::min(fine, std::max(4, 128 / tiles)));
            sp = sp > cap ? cap : sp;
            return sp < 1 ? 1 : sp;
        };
        int cfg;
        if (n % 256 == 0 && ksteps / auto_split(5) >= 24) cfg = 5;
        else cfg = (n % 128 == 0) ? 0 : 1;
        // SwiGLU on 129..256 tiles of 128 columns: un-split, and so fused, where 256 columns would need two K slices
        // and the row kernel (14B gate/up at 8 / 64 / 128 rows 46 / 57 / 66 -> 43 / 50 / 62 us with that kernel)
        if (cfg == 5 && want_epi == EPI_SWIGLU && force_split == 0 && auto_split(5) > 1 && auto_split(0) == 1 && n % 128 == 0) cfg = 0;
        if (cfg == 1 && want_epi == EPI_SWIGLU) want_epi = EPI_PARTIAL;
        const int split = force_split > 0 ? force_split : auto_split(cfg);
        return finish(cfg, split);
    }
    // Above 128 rows no bound decides alone: at a few hundred rows the weight stream, the number of workgroups and the
    // rows a tile pads all count, further up the rounds of tiles over the 256 compute units do.  Time of a launch:
    //   rounds * (fill + slabs * slab) [a partly filled chip runs its slabs up to `part` faster: less traffic, more
    //   clock], not less than the weights take from HBM; a split adds the partial sums written and read back, the row
    //   kernel's own traffic and, if there would be none otherwise, its launch; an un-split residual epilogue adds the
    //   RMSNorm that the row kernel would contain, where one follows.
    // Against the one rule before it (256-row tiles only; slabs through registers on both sides) products of the 7B, 14B and 32B projections and of 24 random
    // shapes at 40 row counts from 129 to 4096 are 1.37 times faster in the mean and more than 3 % slower at a K of six
    // slabs only (7552 columns, 4096 rows: 45 -> 53 us, bound by the stores; the fit holds slabs by the dozen).  The 32B
    // layer's projections take, q/k/v, o, gate/up, down: 573 rows 59 -> 47, 50 -> 47, 395 -> 320, 205 -> 164 us; 300 rows
    // 42 -> 36, 41 -> 36, 272 -> 217, 142 -> 116; 7B at 256 rows 35 -> 19, 38 -> 22, 92 -> 92, 63 -> 53.
    // The bytes of partial sums are bounded by what the workspaces hold, not more tightly: at 48 MiB 7B down of 1200 rows
    // took 2 slices instead of 3 (175 against 161 us) and 32B down of 1280 rows one instead of 5 (378 against 331).
    // Rows of 2^22 values and more take this model at any row count, with as many K slices as fill the chip.  K = 2^22 at
    // 256 columns, 1 / 64 / 128 / 256 / 700 rows: 0.53 / 0.69 / 0.91 / 1.7 / 2.8 ms (un-split on the same tiles 36 / 48 /
    // 68 / 64 / 65; tiles that reach no such rows would take 0.50 / 0.62 / 0.75 up to 128).
    // Time of the partial sums (written and read back) and of the row kernel's own traffic: 11 TB/s while the caches hold
    // them, 5 TB/s in the end (14B o, 4500 rows in two slices, 552 MB: 107 us behind the tiles; 4864 columns, 640 rows in two
    // slices, 62 MB: 4).
    auto moved = [](double b) {
        return (b < 64e6 ? b : 64e6) / 11e6 + (b > 64e6 ? (b < 128e6 ? b - 64e6 : 64e6) / 6e6 : 0.0) + (b > 128e6 ? (b - 128e6) / 5e6 : 0.0);
    };
    const double mn = (double)m * n;
    const double own = want_epi == EPI_RESID ? 8.0 * mn : want_epi == EPI_SWIGLU ? mn : row_kernel ? 2.0 * mn : 4.0 * mn;
    double best = 1e30;
    int best_cfg = -1, best_split = 1, best_rest = 0;
    for (int cfg = 0; cfg < kNumTiles; ++cfg) {
        const TileDef& t = kTiles[cfg];
        // Inside layers the last column tile may reach past n (not on 320 x 256, see DmaTraits), and 192 rows may need more row
        // tiles than 256; products of their own keep to what laps_gemm_plan_info has always reported.  Row kernel included,
        // weights cold, before and with them: 7B gate/up of 200 / 256 rows 77.4 / 82.3 -> 68.6 / 73.9 (198 tiles of 256 x 192
        // where 256 columns make 148), q/k/v of 1847 rows 74.0 -> 68.3, o of 1536 rows 60.1 -> 56.8.
        const bool ragged = n % t.bn != 0;
        if (ragged && (!layer || far || t.bm > 256)) continue;
        if ((cfg == 1 && n % 128 == 0) || (far && cfg != 1 && cfg != 6 && cfg != 7)) continue;
        if (want_epi == EPI_SWIGLU && (cfg == 1 || cfg == 3 || cfg == 4)) continue;   // no gate / up pairs in a wave
        const int tiles_m = (m + t.bm - 1) / t.bm;
        // 320 rows where they need fewer row tiles than 256.  They take in and read from LDS a tenth less per product: 32B
        // gate/up of 280, 640 and 11104 rows 194 -> 156, 334 -> 285 and 4582 -> 4379 us, down of 11104 rows 2405 -> 2238, q/k/v
        // of 1280 rows in two slices 99 -> 76; 206 products of 7B, 14B and 32B at 27 row counts 3 % in the mean.  Products of
        // their own would gain as much; they keep to the 128, 192 or 256 rows that laps_gemm_plan_info has always reported and
        // that its readers rely on.
        if (t.bm == 320 && (!layer || tiles_m == (m + 255) / 256)) continue;
        const bool more_192 = t.bm == 192 && tiles_m != (m + 255) / 256;
        if (more_192 && !layer && !far) continue;
        const double margin = ragged ? kRaggedMargin : more_192 && !far ? kMore192Margin : 1.0;
        const int max_split = force_split > 0 ? force_split : (far ? 256 : 16);   // a few column tiles have to fill the chip
        for (int s = force_split > 0 ? force_split : 1; s <= max_split; ++s) {
            const double partial = 4.0 * s * mn;
            if (force_split == 0 && s > 1 && (ksteps / s < 4 || partial > (double)partial_cap)) break;
            int per = (ksteps + s - 1) / s;
            if (t.ws == 2 && ksteps % 2 == 0) per = (per + 1) / 2 * 2;
            const long wgs = (long)tiles_m * ((n + t.bn - 1) / t.bn) * s;
            const long rounds = (wgs + 255) / 256;
            const double filled = wgs < 256 ? wgs / 256.0 : 1.0;
            const double tiles = 4.0 + rounds * (t.fill + per * t.slab * (1.0 - t.part * (1.0 - filled)));
            const double stream = 4.0 + 2.0 * n * (double)k / 4.6e6;
            double us = (tiles > stream ? tiles : stream) + 0.02 * tiles;   // of equal streams, the one with less to compute
            if (s > 1) us += moved(2.0 * partial + own) + (want_epi == EPI_PARTIAL ? 0.0 : 3.6);
            else if (row_kernel && want_epi == EPI_PARTIAL) us += moved(partial + own);   // written with the tiles
            else if (row_kernel && want_epi == EPI_RESID) us += 4.0 + 6.0 * mn / 4.5e6;
            us *= margin;
            if (us < best) {
                best = us;
                best_cfg = cfg;
                best_split = s;
                best_rest = 0;
            }
            // Whole rounds only, and smaller tiles in one round behind them.
            if (s != 1 || far || ragged || (cfg != 2 && cfg != 10) || wgs <= 256 || wgs % 256 == 0) continue;
            const int columns = mix_columns(tiles_m, n), left = n - columns * 256;
            if (columns < 1) continue;
            for (const MixDef& x : kMix) {
                const int rows = kTiles[x.cfg].bm;
                if ((long)((m + rows - 1) / rows) * ((left + 127) / 128) > 256) continue;
                const double mixed = 4.0 + (wgs / 256) * (t.fill + per * t.slab) + x.fill + per * x.slab;
                const double total = kMixMargin * (us + 1.02 * (mixed > stream ? mixed : stream) - 1.02 * tiles);
                if (tiles > stream && total < best) {
                    best = total;
                    best_cfg = cfg;
                    best_split = 1;
                    best_rest = 1 + x.cfg;
                }
            }
        }
    }
    if (best_cfg < 0) {  // SwiGLU on n % 128 != 0: partial sums of the 64-column panels
        want_epi = EPI_PARTIAL;
        return finish(1, force_split > 0 ? force_split : 1);
    }
    p = finish(best_cfg, best_split);
    p.rest = p.split == 1 ? best_rest : 0;
    return p;
}

size_t laps_gemm_partial_bytes(int m, int n, int k, size_t partial_cap) {   // m <= 128
    // upper bound over the epilogue kinds the layer driver may request
    size_t b = 0;
    for (int e = 0; e < 3; ++e) {
        for (int follows = 0; follows < 2; ++follows) {   // a row kernel
            const GemmPlan p = laps_gemm_plan(m, n, k, 0, e, partial_cap, follows != 0, true);
            const size_t t = p.split > 1 ? (size_t)p.split * m * n * sizeof(float) : 0;
            b = t > b ? t : b;
        }
    }
    // QKV always goes through the partial buffer (its epilogue is a separate kernel)
    const size_t one = (size_t)m * n * sizeof(float);
    return b > one ? b : one;
}

int laps_gemm_launch(const GemmPlan& p, const bf16_t* a, const bf16_t* w, int m, int n, int k, float* out_f32,
                     const float* resid, bf16_t* out_bf16, const int* row_live, const int* n_live, bool live_varies,
                     hipStream_t s) {
    // the last column tile may reach past n where slabs go straight into LDS (DmaTraits::RAGGED)
    const bool ragged_ok = k < kMaxBufferK && n % 64 == 0 && p.cfg >= 0 && p.cfg < kNumTiles && kTiles[p.cfg].bm <= 256;
    if (m < 1 || n < 64 || k < BK || k % BK != 0 || p.cfg < 0 || p.cfg >= kNumTiles || (n % kTiles[p.cfg].bn != 0 && !ragged_ok)) {
        laps_set_error("gemm: unsupported shape m=%d n=%d k=%d for tile %d", m, n, k, p.cfg);
        return LAPS_EINVAL;
    }
    if (p.ws != 1 && (p.k_per_split / BK) % p.ws != 0) {
        laps_set_error("gemm: K slice of %d slabs is not a multiple of the %d weight stages", p.k_per_split / BK, p.ws);
        return LAPS_EINVAL;
    }
    if (!(p.cfg == 1 && p.ws == 1) && p.cfg != 6 && p.cfg != 7 && k >= kMaxBufferK) {
        laps_set_error("gemm: K = %d is too long for tile %d", k, p.cfg);
        return LAPS_EINVAL;
    }
    if (p.epi != EPI_PARTIAL && p.split != 1) {
        laps_set_error("gemm: fused epilogue needs a single K slice");
        return LAPS_EINVAL;
    }
    GemmArgs g;
    g.A = a;
    g.W = w;
    g.M = m;
    g.N = n;
    g.K = k;
    g.split = p.split;
    g.kps = p.k_per_split;
    g.tiles_m = (m + kTiles[p.cfg].bm - 1) / kTiles[p.cfg].bm;
    g.tiles_n = (n + kTiles[p.cfg].bn - 1) / kTiles[p.cfg].bn;
    g.out_f32 = out_f32;
    g.resid = resid;
    g.out_bf16 = out_bf16;
    g.row_live = row_live;
    g.n_live = n_live;
    g.cols = n;
    // Loads straight into LDS are given 16-byte pieces that lie on 16-byte bounds: rows are whole multiples of 128 bytes, so
    // the bases decide.  (5120 x 5120 at 8 / 128 / 2048 rows, weights cold: 22 / 25 / 92 us, with weights 2 bytes off 26 / 30 / 155.)
    const bool aligned = ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(w)) & 15) == 0;
    // batches of an unknown number of live rows, un-split plans of the tiles of one workgroup a unit: chosen on the device
    if (aligned && live_varies && n_live && m > 256 && k < kMaxBufferK && p.split == 1 && kTiles[p.cfg].bm >= 192 && p.cfg != 7 && n % 256 == 0) {
        if (p.epi == EPI_PARTIAL) return launch_live<EPI_PARTIAL>(g, s);
        if (p.epi == EPI_RESID) return launch_live<EPI_RESID>(g, s);
        return launch_live<EPI_SWIGLU>(g, s);
    }
    if (p.rest != 0 && aligned && k < kMaxBufferK) {
        int small = -1;
        for (int i = 0; i < 3; ++i)
            if (kMix[i].cfg == p.rest - 1) small = i;
        if (small < 0 || (p.cfg != 2 && p.cfg != 10) || p.split != 1 || n % 256 != 0 || mix_columns(g.tiles_m, n) < 1 ||
            mix_columns(g.tiles_m, n) >= n / 256) {
            laps_set_error("gemm: no tile %d behind whole rounds of tile %d (m=%d n=%d)", p.rest - 1, p.cfg, m, n);
            return LAPS_EINVAL;
        }
        if (p.epi == EPI_PARTIAL) return launch_mix<EPI_PARTIAL>(g, p.cfg == 10, small, s);
        if (p.epi == EPI_RESID) return launch_mix<EPI_RESID>(g, p.cfg == 10, small, s);
        return launch_mix<EPI_SWIGLU>(g, p.cfg == 10, small, s);
    }
    if (k >= kMaxBufferK || !aligned) {
        int cfg = p.cfg, ws = p.ws;
        if (k < kMaxBufferK) {   // the plan's K slices on the widest pointer-addressed tile that fills the chip or divides n
            const bool wide = n % 256 == 0 && (long)((m + 191) / 192) * (n / 256) * p.split >= 256;
            cfg = wide ? 6 : n % 128 == 0 ? 7 : 1;
            ws = 1;
            g.tiles_m = (m + kTiles[cfg].bm - 1) / kTiles[cfg].bm;
            g.tiles_n = n / kTiles[cfg].bn;
        }
        if (cfg == 1 && p.epi == EPI_SWIGLU) return launch_far<128, 64, 4, 1, EPI_SWIGLU, 1>(g, s);   // pairs in a wave of 64 columns
#define LAPS_FAR_CASE(cfg, BM, BN, WS)                                                          \
    case (cfg) * 8 + (WS):                                                                      \
        if (p.epi == EPI_PARTIAL) return launch_far<BM, BN, 2, 2, EPI_PARTIAL, WS>(g, s);       \
        if (p.epi == EPI_RESID) return launch_far<BM, BN, 2, 2, EPI_RESID, WS>(g, s);           \
        if constexpr (BN % 128 == 0) return launch_far<BM, BN, 2, 2, EPI_SWIGLU, WS>(g, s);     \
        break
        switch (cfg * 8 + ws) {
            LAPS_FAR_CASE(1, 128, 64, 1);
            LAPS_FAR_CASE(6, 192, 256, 1);
            LAPS_FAR_CASE(6, 192, 256, 2);
            LAPS_FAR_CASE(7, 192, 128, 1);
            default: break;
        }
#undef LAPS_FAR_CASE
    } else {
        // Weights that one row tile reads alone bypass the caches (32B, 128 rows: gate/up 114 us through them, 104 bypassing,
        // down 64 and 54, q/k/v 21.8 and 21.0); several row tiles that share them lose by it (2048 rows, q/k/v 109 cached, 116
        // bypassing).  A product of its own (no batch whose live rows are given) may find its weights in the memory-side cache
        // the next time: where that holds them and K is split over narrow tiles, they stay in the caches above 48 rows (weights
        // cold / warm, cached against bypassing: 14B down 48 rows 32.9 / 29.2 against 30.9 / 30.2, 64 rows 33.9 / 29.9 against
        // 32.7 / 32.0, 128 rows 39.7 / 32.3 against 40.0 / 40.1, 160 rows 42.5 / 33.8 against 42.5 / 42.7; o 128 rows 23.2 / 18.8
        // against 25.1 / 25.0; 32B down of 283 MB, 160 rows 74.7 against 68.8).
        const bool alone = row_live == nullptr && n_live == nullptr;
        const bool keep = alone && m > 48 && p.split > 1 && kTiles[p.cfg].bn < 256 && 2.0 * n * k <= 256e6;
        const bool bypass = g.tiles_m == 1 && !keep;
#define LAPS_DMA_CASE(cfg, BM, BN, WM, WN)                                                       \
    case cfg:                                                                                    \
        if (bypass) return launch_dma_epi<BM, BN, WM, WN, true>(p.epi, g, s);                    \
        return launch_dma_epi<BM, BN, WM, WN, false>(p.epi, g, s)
        // Up to 64 rows the tiles of 64 rows spare the LDS reads and the products of as many rows of nothing.  65 to 128 rows are
        // two of them where 128 columns leave compute units for twice the workgroups: a unit takes in 64 rows of A beside the
        // weights instead of 128.  Through registers / 128 rows this way / 64: 2560 x 1024 at 80 / 128 rows 12.1 / 12.1 / 10.0 and
        // 13.3 / 14.5 / 11.1 us, 3584 x 3584 in 4 slices, 128 rows, 18.6 / 18.8 / 15.9, 14336 x 1024 14.3 / 14.9 / 12.1.
        if (p.cfg == 0 && m > 64 && m <= 128 && 2 * g.tiles_n * p.split <= 256) {
            g.tiles_m = 2;
            return launch_dma_epi<64, 128, 2, 2, false>(p.epi, g, s);
        }
        if (m <= 64) switch (p.cfg) {
            LAPS_DMA_CASE(0, 64, 128, 2, 2);
            LAPS_DMA_CASE(5, 64, 256, 1, 4);
            default: break;
        }
        switch (p.cfg) {
            LAPS_DMA_CASE(0, 128, 128, 2, 2);
            LAPS_DMA_CASE(1, 128, 64, 2, 2);
            LAPS_DMA_CASE(2, 256, 256, 2, 2);
            LAPS_DMA_CASE(3, 256, 224, 4, 1);
            LAPS_DMA_CASE(4, 256, 160, 4, 1);
            LAPS_DMA_CASE(5, 128, 256, 1, 4);
            LAPS_DMA_CASE(6, 192, 256, 2, 2);
            LAPS_DMA_CASE(7, 192, 128, 2, 2);
            LAPS_DMA_CASE(8, 256, 128, 2, 2);
            LAPS_DMA_CASE(9, 256, 192, 4, 1);
            LAPS_DMA_CASE(10, 320, 256, 2, 2);
            default: break;
        }
#undef LAPS_DMA_CASE
    }
    laps_set_error("gemm: no kernel for tile %d with epilogue %d", p.cfg, p.epi);
    return LAPS_EINVAL;
}
