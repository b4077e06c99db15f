// Ragged, paged, causal grouped-query flash attention for gfx950.
//
// One workgroup = one (sequence, kv head, block of query rows).  A "query row" is a (new token t,
// query head g of the kv head's group) pair, numbered r = t*G + g, so the G query heads that share a
// kv head are packed into the MFMA row dimension and every K/V page is fetched once for all of them.
// The workgroup walks the sequence's pages (cached prefix first, then the new tokens, which the QKV
// step has already appended) in tiles of 64 keys: coalesced 4 KB page reads -> registers -> LDS.
//
// Both products are issued transposed so that a lane owns one query row end to end:
//   S^T = K Q^T   (A = K fragment from LDS, B = Q fragment held in registers)
//   O^T = V^T P^T (A = V^T fragment from LDS - V pages are stored [head_dim][16 tokens], B = P)
// With the 32x32 accumulator layout (lane -> column, registers -> rows) the softmax statistics of a
// row live in one lane and its partner lane^32: row max and row sum need a single cross-lane
// exchange, and the O rescale is a per-lane scalar.  K rows are read from LDS through the
// permutation key(8a + 4h + b) = 16(a/2) + 8h + 4(a%2) + b, which makes the eight probabilities a
// lane holds in accumulator registers 8u..8u+7 exactly the eight consecutive keys its P fragment
// must supply to the second product - no shuffles between the two MFMA stages.
//
// Two loops share these pieces.  Workgroups of 4 waves (short prompts, split key ranges) take a tile at a time:
// scores, softmax, second product, one barrier.  Workgroups of 8 waves (long prompts) run a three-stage software
// pipeline over 32-key half tiles, in which the matrix cores work on the half tiles before and after the one whose
// softmax the vector ALU is computing; its row sums also come from the matrix cores.  In both, the value the
// exponentials subtract follows the row maximum lazily, so that O is rescaled rarely.
//
// Few query rows over a long cached prefix (a short re-prefill turn) would leave most of the chip idle:
// one request of 16 new tokens is a single row block per kv head.  For such launches the key range of
// each row block is split into parts of equal length (laps_dev_attn_desc; at least 4 key tiles each, or one
// where few workgroups make it pay); every part writes its un-normalised accumulator with its running maximum
// and row sum, and a second kernel merges the parts of a block in key order, so the result depends neither on
// scheduling nor on the lengths of other sequences.  The number of workgroups is a function of launch shapes only
// (row blocks, kv heads, page-table width), which keeps captured graphs replayable; how many of the parts a
// block really has is worked out on the device from its length.
//
// Many query rows over page tables that allow long prefixes (chunks of long prompts, mixed batches, groups of turns) make
// blocks of very different lengths.  Such launches run the 8-wave loop in a fixed number of workgroups, each of which walks
// an equal share of the batch's (kv head, row block) units, worked out on the device from the batch's lengths; a unit cut
// between shares leaves partial results like a split key range, merged in key order by a kernel of its own.
#include "laps_internal.h"

#include <climits>
#include <type_traits>

namespace {

constexpr int KT = LAPS_ATTN_KT;   // keys per tile (4 pages)

__device__ __forceinline__ int swz8(int row, int c) { return c ^ ((row & 7) ^ ((row >> 3) & 1)); }
__device__ __forceinline__ int swz16(int row, int c) { return c ^ (row & 15); }

// NW waves per workgroup, one 32-row query tile per wave: rows per workgroup = 32 * NW.  With NW = 8
// two waves share a SIMD, so one wave's softmax (VALU, exp) overlaps the other's MFMAs.
constexpr int MIN_TILES_PER_SPLIT = 4;   // key tiles per part of a split key range (lower bound, attn_blocking)

// Two waves per SIMD in every variant (second launch-bound argument): with 4 waves per workgroup that is two
// resident workgroups per compute unit, which the key-streaming launches need to cover the memory latency.
// HALVES: the 4-wave loop forms its probabilities and row sums by half tiles, as the 8-wave loop does: the same bits.
// PERSIST: a fixed number of workgroups, each walking its share of the batch (laps_dev_attn_bounds); a share may begin
// and end inside a unit, whose parts then go through partial results like the splits.
template <int HD, int NW, bool SPLIT, bool PERSIST, bool HALVES = false>
__global__ __launch_bounds__(NW * 64, 2) void attn_kernel(const bf16_t* __restrict__ q, bf16_t* __restrict__ out,
                                                        float* __restrict__ part_o, float* __restrict__ part_ml,
                                                        const bf16_t* __restrict__ k_pool,
                                                        const bf16_t* __restrict__ v_pool,
                                                        const int4* __restrict__ desc,
                                                        const int* __restrict__ page_table, int max_pages,
                                                        const int* __restrict__ tile_start, int n_seq, int n_q,
                                                        int n_kv, float scale_log2e, int n_pool_pages, int n_tokens,
                                                        int max_items, const int4* __restrict__ bounds) {
    constexpr int NTHR = NW * 64;
    constexpr int CPR = HD / 8;            // 16-byte chunks per K row
    constexpr int CPP = HD * 2;            // 16-byte chunks per page (K and V alike)
    constexpr int NLD = KT * CPR / NTHR;   // chunk loads per thread per tile, K and V each
    constexpr int KSTEPS = HD / 16;        // MFMA k-steps over head_dim
    constexpr int NI = HD / 32;            // output sub-tiles over head_dim
    constexpr int ROWS = 32 * NW;
    static_assert(KT * CPR % NTHR == 0, "tile chunks must divide over the threads");

    __shared__ __align__(16) u32x4 Ks[2][KT * CPR];   // double buffered: one barrier per tile
    __shared__ __align__(16) u32x4 Vs[2][HD * 8];

    const int G = n_q / n_kv;
    // one unit: (item, kv head), key tiles [t0, t1) of it if PERSIST; slot: where a cut unit's result goes
    auto unit = [&](const int item, const int kvh, const int t0, const int t1, const int slot) __attribute__((always_inline)) {
    const int4 it = desc[2 * item];
    const int4 at = desc[2 * item + 1];
    const int seq = it.x, qtile = it.y, L = it.z, H = it.w, rs = at.x;
    if (seq < 0) return;
    // row offsets come from the caller's device array: rows outside the batch are never touched, whatever it holds
    if (rs < 0 || L > n_tokens - rs) return;
    const int n_rows = L * G;
    const int kv_len = H + L;
    // never index past the table's width, whatever the lengths say (keys beyond it then repeat the last page)
    const int n_pages_need = (kv_len + LAPS_PAGE - 1) / LAPS_PAGE;
    const int n_pages_seq = n_pages_need < max_pages ? n_pages_need : max_pages;
    const int R0 = qtile * ROWS;
    if (R0 >= n_rows) return;
    const int last_row_wg = (R0 + ROWS < n_rows ? R0 + ROWS : n_rows) - 1;
    const int kv_end_all = H + last_row_wg / G + 1;  // keys visible to the last row of this block
    int kv_begin = 0, kv_end = kv_end_all;
    if (SPLIT) {
        if ((int)blockIdx.z >= at.y) return;   // the item has fewer parts
        kv_begin = blockIdx.z * at.z * KT;
        kv_end = kv_begin + at.z * KT < kv_end_all ? kv_begin + at.z * KT : kv_end_all;
    }
    if (PERSIST) {
        kv_begin = t0 * KT;
        kv_end = t1 < (kv_end_all + KT - 1) / KT ? t1 * KT : kv_end_all;
    }
    const bool whole = SPLIT ? at.y == 1 : (!PERSIST || (kv_begin == 0 && kv_end == kv_end_all));
    const int* pt = page_table + (size_t)seq * max_pages;
    const size_t tok0 = (size_t)rs;
    const int q_stride = n_q * HD;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lm = lane & 31, lh = lane >> 5;

    // ---- this wave's 32 query rows: Q fragments stay in registers for the whole kernel
    const int base = R0 + wave * 32;
    const int row_id = base + lm;
    const int rc = row_id < n_rows ? row_id : n_rows - 1;
    const int tq = rc / G, gq = rc - tq * G;
    const int limit = H + tq;                                        // last visible key of this lane's row
    const int vis_min = H + (base < n_rows ? base : n_rows - 1) / G;  // wave-uniform: every row sees keys <= vis_min
    const int vis_max = (base < n_rows) ? H + (base + 31 < n_rows ? base + 31 : n_rows - 1) / G : -1;
    bf16x8 qf[KSTEPS];
    {
        const u32x4* qp = reinterpret_cast<const u32x4*>(q + (tok0 + tq) * q_stride + (size_t)(kvh * G + gq) * HD);
#pragma unroll
        for (int kk = 0; kk < KSTEPS; ++kk) qf[kk] = __builtin_bit_cast(bf16x8, qp[kk * 2 + lh]);
    }
    f32x16 o[NI];
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[ni][i] = 0.f;
    float m_run = -INFINITY, l_run = 0.f;   // running max (in log2 units, already scaled) and partial row sum

    // ---- tile copy assignment: chunk c = tid + i*NTHR of the tile's 4 pages.  All chunks a wave copies in one
    // pass lie in one page, so the page id is a wave-uniform (scalar) load.
    u32x4 kreg[NLD], vreg[NLD];   // landing registers of the tile copy
    auto page_id = [&](int j0, int i) -> int {
        int pidx = j0 / LAPS_PAGE + __builtin_amdgcn_readfirstlane((tid + i * NTHR) / CPP);
        pidx = pidx < n_pages_seq ? pidx : n_pages_seq - 1;  // past the end: any valid page, masked later
        return pt[pidx];
    };
    auto chunk_offset = [&](int pg, int i) -> size_t {
        const int within = (tid + i * NTHR) % CPP;
        // an unset (-1) entry or an id outside the pool must not turn into a wild address
        const size_t page = (size_t)((pg > 0 && pg < n_pool_pages) ? pg : 0);
        return (page * n_kv + kvh) * CPP + within;
    };
    auto store_k = [&](int buf) {   // K page is [16 keys][HD]
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int c = tid + i * NTHR;
            const int pi = c / CPP, within = c % CPP;
            const int key = pi * LAPS_PAGE + within / CPR, kc = within % CPR;
            Ks[buf][key * CPR + (CPR == 16 ? swz16(key, kc) : swz8(key, kc))] = kreg[i];
        }
    };
    auto store_v = [&](int j0, int buf) {   // V page is [HD][16 keys]: chunk = 8 consecutive keys of one head_dim index
        const bool tail = (j0 + KT > kv_len);
#pragma unroll
        for (int i = 0; i < NLD; ++i) {
            const int c = tid + i * NTHR;
            const int pi = c / CPP, within = c % CPP;
            const int e = within / 2, half = within & 1;
            u32x4 v = vreg[i];
            if (tail) {  // zero keys >= kv_len so that 0 * garbage cannot produce NaN
                const int nvalid = kv_len - (j0 + pi * LAPS_PAGE + half * 8);
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    unsigned x = v[w];
                    if (2 * w + 1 >= nvalid) x &= 0x0000ffffu;
                    if (2 * w >= nvalid) x = 0u;
                    v[w] = x;
                }
            }
            Vs[buf][e * 8 + swz8(e, pi * 2 + half)] = v;
        }
    };

    // MFMA row rho = lm of the first product holds key 16(a/2) + 8h + 4(a%2) + b with rho = 8a + 4h + b
    const int ra = lm >> 3, rh = (lm >> 2) & 1, rb = lm & 3;
    const int krow = 16 * (ra >> 1) + 8 * rh + 4 * (ra & 1) + rb;

    // operand fragments: K for matrix instruction g = 2 kk + sub of the first product, V^T for g = NI u2 + ni of
    // the second
    auto k_frag = [&](int kb, int g) -> bf16x8 {
        const int row = (g & 1) * 32 + krow, ch = (g >> 1) * 2 + lh;
        return __builtin_bit_cast(bf16x8, Ks[kb][row * CPR + (CPR == 16 ? swz16(row, ch) : swz8(row, ch))]);
    };
    auto v_frag = [&](int vb, int g) -> bf16x8 {
        const int row = (g % NI) * 32 + lm;
        return __builtin_bit_cast(bf16x8, Vs[vb][row * 8 + swz8(row, (g / NI) * 2 + lh)]);
    };
    // S^T = K Q^T for the 64 keys of the tile in Ks[kb] (two 32-key sub-tiles)
    auto qk_tile = [&](int kb, f32x16 (&s)[2]) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int i = 0; i < 16; ++i) s[sub][i] = 0.f;
#pragma unroll
        for (int g = 0; g < 2 * KSTEPS; ++g)
            s[g & 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(kb, g), qf[g >> 1], s[g & 1], 0, 0, 0);
    };
    // causal mask, needed on diagonal tiles only (wave-uniform test by the caller)
    auto mask_tile = [&](int j0, f32x16 (&s)[2]) {
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const int a = i >> 2, b = i & 3;
                const int key = j0 + sub * 32 + 16 * (a >> 1) + 8 * lh + 4 * (a & 1) + b;
                s[sub][i] = (key <= limit) ? s[sub][i] : -INFINITY;
            }
    };
    // online softmax of one tile's scores, one query row per lane (shared with lane^32): probabilities as the
    // second product's operand, the tile's row maximum and row sum; softmax_finish folds them into the running
    // state and rescales O when some row's maximum moved
    // The reference value m_run that the exponentials subtract follows the row maximum lazily: it moves (and O and
    // the row sum are rescaled) only when some row's maximum has grown by more than RESCALE_SLACK in log2 units, so
    // probabilities stay below 2^RESCALE_SLACK and the 64-register rescale of O is rare.  The quotient O / l does
    // not depend on the reference.
    constexpr float RESCALE_SLACK = 8.f;
    const int partner_addr = (lane ^ 32) << 2;   // ds_bpermute address of the lane that shares this lane's row
    auto from_partner = [&](float x) {
        return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(partner_addr, __builtin_bit_cast(int, x)));
    };
    float m_new, psum;
    bool moved;   // wave-uniform: the reference moves to m_new after this tile
    auto pick_reference = [&](float mx) -> float {   // returns what this tile's exponentials subtract
        m_new = fmaxf(m_run, mx * scale_log2e);
        moved = __builtin_amdgcn_ballot_w64(m_new > m_run + RESCALE_SLACK) != 0;
        const float m_use = moved ? m_new : m_run;
        // un-split: finite from the first tile on (key 0 is visible to every row).  A later split can start
        // on a diagonal tile in which a row sees nothing yet: keep exp2(-inf - -inf) out of the arithmetic.
        return (SPLIT && m_use == -INFINITY) ? 0.f : m_use;
    };
    auto softmax_tile = [&](f32x16 (&s)[2], bf16x8 (&pf)[2][2]) {
        float mx = -INFINITY;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, s[sub][i]);
        mx = fmaxf(mx, from_partner(mx));
        const float m_sub = pick_reference(mx);
        psum = 0.f;
#pragma unroll
        for (int sub = 0; sub < 2; ++sub)
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 pk;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[sub][8 * u + e], scale_log2e, -m_sub));
                    psum += p;
                    pk[e] = (__bf16)p;
                }
                pf[sub][u] = pk;
            }
    };
    auto softmax_finish = [&]() {
        if (moved) {
            const float alpha = (SPLIT && m_new == -INFINITY) ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[ni][i] *= alpha;
            m_run = m_new;
        }
        l_run += psum;
    };
    // O^T += V^T P^T with the tile in Vs[vb]
    auto pv_tile = [&](int vb, bf16x8 (&pf)[2][2]) {
#pragma unroll
        for (int g = 0; g < 4 * NI; ++g)
            o[g % NI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(vb, g), pf[g / (2 * NI)][(g / NI) & 1], o[g % NI], 0, 0, 0);
    };

    // the same by half tiles of 32 keys (the 8-wave loop, HALVES)
    [[maybe_unused]] auto mask_half = [&](int j0, int h, f32x16& sc) {
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int a = i >> 2, b = i & 3;
            const int key = j0 + h * 32 + 16 * (a >> 1) + 8 * lh + 4 * (a & 1) + b;
            sc[i] = (key <= limit) ? sc[i] : -INFINITY;
        }
    };
    // Row sums come from the matrix cores as well: a fragment of ones times P^T gives, in every register of the
    // result, the sum over the fragment's keys of the probabilities as the second product sees them (rounded to
    // bf16), complete in both lanes of a row.  It is added to l_run where the same probabilities are added to O.
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
    [[maybe_unused]] auto softmax_half = [&](f32x16& sc, bf16x8 (&pf)[2]) {
        float mx = -INFINITY;
#pragma unroll
        for (int i = 0; i < 16; ++i) mx = fmaxf(mx, sc[i]);
        mx = fmaxf(mx, from_partner(mx));
        const float m_sub = pick_reference(mx);
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            bf16x8 pk;
#pragma unroll
            for (int e = 0; e < 8; ++e)
                pk[e] = (__bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[8 * u + e], scale_log2e, -m_sub));
            pf[u] = pk;
        }
    };
    [[maybe_unused]] auto pv_half = [&](int vb, int h, bf16x8 (&pf)[2]) {
#pragma unroll
        for (int g = 0; g < 2 * NI; ++g)
            o[g % NI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_frag(vb, (2 * h + g / NI) * NI + g % NI), pf[g / NI],
                                                                o[g % NI], 0, 0, 0);
        f32x16 ls;
#pragma unroll
        for (int i = 0; i < 16; ++i) ls[i] = 0.f;
        ls = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pf[0], ls, 0, 0, 0);
        ls = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pf[1], ls, 0, 0, 0);
        l_run += ls[0];
    };
    // moves the reference to m_new after the matrix work of a half step (the probabilities just formed already
    // use it; O and l_run, which hold the half tiles before, follow here)
    [[maybe_unused]] auto move_reference = [&]() {
        if (moved) {
            const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);
            l_run *= alpha;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int i = 0; i < 16; ++i) o[ni][i] *= alpha;
            m_run = m_new;
        }
    };

    const auto exists = [&](int j) { return j < kv_end; };
    if constexpr (NW == 8) {
        // Long prompts.  The loop is software-pipelined three deep over 32-key half tiles: in step w the matrix
        // cores form the scores of half tile w + 1 and add half tile w - 1 to O while the vector ALU turns the scores
        // of half tile w into probabilities - one matrix instruction, one LDS fragment read and a share of the
        // softmax per slot, so both pipes are busy in every wave whatever phase the other wave of its SIMD is in.
        // Tile t occupies Ks[t&1] and Vs[t&1].  Tile step t runs the half steps 2t and 2t + 1:
        //   2t    : scores of (t, keys 32..63), softmax of (t, keys 0..31), O += (t-1, keys 32..63)
        //   barrier: K(t) and V(t-1) are done with; K(t+2) and V(t+1) leave the registers for their buffers
        //   2t + 1: scores of (t+1, keys 0..31), softmax of (t, keys 32..63), O += (t, keys 0..31)
        // and there is one tile step more than tiles (its first half adds the last half tile to O).
        // page ids (scalars) are fetched one tile step before the loads that use them
        int idk[NLD], idv[NLD];
        auto fetch_ids = [&](int jk, int jv) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) idk[i] = page_id(jk, i), idv[i] = page_id(jv, i);
        };
        auto load_k = [&]() {
#pragma unroll
            for (int i = 0; i < NLD; ++i) kreg[i] = reinterpret_cast<const u32x4*>(k_pool)[chunk_offset(idk[i], i)];
        };
        auto load_v = [&]() {
#pragma unroll
            for (int i = 0; i < NLD; ++i) vreg[i] = reinterpret_cast<const u32x4*>(v_pool)[chunk_offset(idv[i], i)];
        };
        // wave-uniform: half tile (tile at key j, half h) exists and some row of this wave sees one of its keys
        const auto visible = [&](int j, int h) { return j >= kv_begin && j < kv_end && j + 32 * h <= vis_max; };
        constexpr int NQ = KSTEPS;       // matrix instructions of each product per half tile (equal: HD / 16)
        constexpr int NS = 2 * NQ;       // slots per half step
        constexpr int MAXS = NS >= 16 ? NS / 8 : 1;   // slots that take the row maximum
        constexpr int EXP0 = MAXS + 2;   // first slot of the exponentials
        constexpr int NE = NS + 2 - EXP0;   // slots that share the 16 exponentials
        static_assert(2 * NI == NQ, "both products issue HD / 16 matrix instructions per half tile");
        // the three stages one after the other, for the first and last half steps of a wave
        auto qk_half = [&](int kb, int h, f32x16& sc) {
#pragma unroll
            for (int i = 0; i < 16; ++i) sc[i] = 0.f;
#pragma unroll
            for (int kk = 0; kk < KSTEPS; ++kk)
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_frag(kb, 2 * kk + h), qf[kk], sc, 0, 0, 0);
        };
        // one half step.  (kb, hq): buffer and half of the scores to form into s_nxt; s_cur -> pf_cur; (vb, hv):
        // buffer and half of the V tile that goes with pf_prev
        auto half_step = [&](bool do_qk, bool do_sm, bool do_pv, int kb, int hq, f32x16& s_nxt, f32x16& s_cur,
                             bf16x8 (&pf_cur)[2], int vb, int hv, bf16x8 (&pf_prev)[2]) __attribute__((always_inline)) {
            if (do_qk && do_sm && do_pv) {
                // slot g < NS: even = first product's instruction g / 2, odd = second product's; the last two slots
                // take the row sums.  The LDS fragment of slot g + 2 is read in slot g.
                bf16x8 fr[NS + 2];
                fr[0] = k_frag(kb, hq);
                fr[1] = v_frag(vb, 2 * hv * NI);
                f32x16 ls;
#pragma unroll
                for (int i = 0; i < 16; ++i) s_nxt[i] = 0.f, ls[i] = 0.f;
                float cmax[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
                float mx = 0.f, mx_other = 0.f, m_sub = 0.f;
                bf16x8 pk;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int g = 0; g < NS + 2; ++g) {
                    const int q = g >> 1;   // index within its product
                    if (g >= NS)
                        ls = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ones, pf_prev[g - NS], ls, 0, 0, 0);
                    else if (g & 1)
                        o[q % NI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g], pf_prev[q / NI], o[q % NI], 0, 0, 0);
                    else
                        s_nxt = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[g], qf[q], s_nxt, 0, 0, 0);
                    if (g + 2 < NS) {
                        const int q2 = (g + 2) >> 1;
                        fr[g + 2] = ((g + 2) & 1) ? v_frag(vb, (2 * hv + q2 / NI) * NI + q2 % NI) : k_frag(kb, 2 * q2 + hq);
                    }
                    // ---- this slot's share of the softmax
                    if (g < MAXS) {   // four independent chains over 16 / MAXS values per slot
                        constexpr int PER = 16 / MAXS;
#pragma unroll
                        for (int k = 0; k < PER; ++k) cmax[k & 3] = fmaxf(cmax[k & 3], s_cur[g * PER + k]);
                    } else if (g == MAXS) {
                        mx = fmaxf(fmaxf(cmax[0], cmax[1]), fmaxf(cmax[2], cmax[3]));
                        mx_other = from_partner(mx);
                    } else if (g == MAXS + 1) {
                        m_sub = pick_reference(fmaxf(mx, mx_other));
                    } else {
#pragma unroll
                        for (int k = 0; k < 16; ++k) {
                            if ((k * NE) / 16 != g - EXP0) continue;
                            float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s_cur[k], scale_log2e, -m_sub));
                            asm volatile("" : "+v"(p));   // keeps the exponential in its slot (it would sink below
                                                          // the rescale branch, out from under the matrix work)
                            pk[k & 7] = (__bf16)p;
                            if ((k & 7) == 7) pf_cur[k >> 3] = pk;
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                l_run += ls[0];
                move_reference();
            } else {
                if (do_qk) qk_half(kb, hq, s_nxt);
                if (do_sm) softmax_half(s_cur, pf_cur);
                if (do_pv) pv_half(vb, hv, pf_prev);
                if (do_sm) move_reference();
            }
        };
        f32x16 s_lo, s_hi;            // scores of keys 0..31 / 32..63 of a tile
        bf16x8 p_lo[2], p_hi[2];      // their probabilities
        auto tile_step = [&](int j0, auto parity) __attribute__((always_inline)) {
            constexpr int b = decltype(parity)::value;   // j0's tile sits in buffers b, its neighbours in b ^ 1
            {
                const bool sm = visible(j0, 0);
                if (sm && j0 + 31 > vis_min) mask_half(j0, 0, s_lo);
                half_step(visible(j0, 1), sm, visible(j0 - KT, 1), b, 1, s_hi, s_lo, p_lo, b ^ 1, 1, p_hi);
            }
            __syncthreads();
            if (exists(j0 + 2 * KT)) store_k(b);
            if (exists(j0 + KT)) store_v(j0 + KT, b ^ 1);
            if (exists(j0 + 3 * KT)) load_k();
            if (exists(j0 + 2 * KT)) load_v();
            fetch_ids(j0 + 4 * KT, j0 + 3 * KT);   // clamped to the sequence's pages: harmless past the end
            {
                const bool sm = visible(j0, 1);
                if (sm && j0 + 63 > vis_min) mask_half(j0, 1, s_hi);
                half_step(visible(j0 + KT, 0), sm, visible(j0, 0), b ^ 1, 0, s_lo, s_hi, p_hi, b, 0, p_lo);
            }
        };
        // SPLIT is never combined with this variant: a wave's first half tile always shows a key to every row (key 0,
        // or the first key after a cut, which laps_dev_attn_bounds places where all rows see it), so the running
        // maximum is finite from the first softmax on
        static_assert(!SPLIT, "the pipelined loop serves un-split launches only");
        if (PERSIST) __syncthreads();   // the unit before is done with the LDS tiles
        fetch_ids(kv_begin, kv_begin);
        load_k();
        load_v();
        fetch_ids(kv_begin + KT, kv_begin + KT);
        store_k(0);
        store_v(kv_begin, 0);
        if (exists(kv_begin + KT)) load_k();
        fetch_ids(kv_begin + 2 * KT, kv_begin + KT);
        __syncthreads();
        if (visible(kv_begin, 0)) qk_half(0, 0, s_lo);
        if (exists(kv_begin + KT)) store_k(1);
        if (exists(kv_begin + 2 * KT)) load_k();
        if (exists(kv_begin + KT)) load_v();
        fetch_ids(kv_begin + 3 * KT, kv_begin + 2 * KT);
        for (int j0 = kv_begin; j0 < kv_end + KT; j0 += 2 * KT) {   // two tile steps: the buffers swap roles
            tile_step(j0, std::integral_constant<int, 0>{});
            if (j0 + KT < kv_end + KT) tile_step(j0 + KT, std::integral_constant<int, 1>{});
        }
    } else {
        // Short prompts and key-range splits: a few tiles per workgroup, latency matters more than overlap.  The
        // page ids of a tile are fetched one step before its data, so that the two dependent loads (table entry,
        // then the page itself) do not add up on the critical path of every tile.
        int pgn[NLD];
        auto load_pages = [&](int j0) {
#pragma unroll
            for (int i = 0; i < NLD; ++i) pgn[i] = page_id(j0, i);
        };
        auto load_tile = [&]() {   // uses the ids load_pages fetched
#pragma unroll
            for (int i = 0; i < NLD; ++i) {
                const size_t off = chunk_offset(pgn[i], i);
                kreg[i] = reinterpret_cast<const u32x4*>(k_pool)[off];
                vreg[i] = reinterpret_cast<const u32x4*>(v_pool)[off];
            }
        };
        load_pages(kv_begin);
        load_tile();
        load_pages(kv_begin + KT);        // indices are clamped to the sequence's pages: harmless past the end
        store_k(0);
        store_v(kv_begin, 0);
        if (exists(kv_begin + KT)) {
            load_tile();
            load_pages(kv_begin + 2 * KT);
        }
        __syncthreads();
        int buf = 0;
        for (int j0 = kv_begin; j0 < kv_end; j0 += KT, buf ^= 1) {
            // stage the next tile (already in registers) into the other buffer, refill the registers
            if (exists(j0 + KT)) {
                store_k(buf ^ 1);
                store_v(j0 + KT, buf ^ 1);
                if (exists(j0 + 2 * KT)) {
                    load_tile();
                    load_pages(j0 + 3 * KT);
                }
            }
            if (j0 <= vis_max) {  // wave-uniform: something of this tile is visible to this wave
                f32x16 sc[2];
                bf16x8 pf[2][2];
                qk_tile(buf, sc);
                if constexpr (HALVES) {
#pragma unroll
                    for (int h = 0; h < 2; ++h) {
                        if (j0 + 32 * h > vis_max) continue;
                        if (j0 + 32 * h + 31 > vis_min) mask_half(j0, h, sc[h]);
                        softmax_half(sc[h], pf[h]);
                        move_reference();
                        pv_half(buf, h, pf[h]);
                    }
                } else {
                    if (j0 + KT - 1 > vis_min) mask_tile(j0, sc);
                    softmax_tile(sc, pf);
                    softmax_finish();
                    pv_tile(buf, pf);
                }
            }
            __syncthreads();
        }
    }

    // ---- normalise and store: lane owns row r; register i of sub-tile ni is head_dim index
    //      ni*32 + 8*(i/4) + 4*(lane/32) + i%4
    // row sums by half tiles are complete, the plain loop's are a lane's share
    const float l_tot = (NW == 8 || HALVES) ? l_run : l_run + __shfl_xor(l_run, 32, 64);
    if (!whole) {
        // partial result of this key range: accumulator as [4-float chunk][row] so that the 32 rows of a half
        // wave write consecutive 16-byte pieces; (running max, row sum) per row
        if (row_id < n_rows) {
            const size_t blk = PERSIST ? (size_t)slot : ((size_t)item * n_kv + kvh) * gridDim.z + blockIdx.z;
            const int row = wave * 32 + lm;
            f32x4* po = reinterpret_cast<f32x4*>(part_o) + blk * (size_t)(HD / 4) * ROWS;
#pragma unroll
            for (int ni = 0; ni < NI; ++ni)
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    f32x4 w;
                    w.x = o[ni][4 * a]; w.y = o[ni][4 * a + 1]; w.z = o[ni][4 * a + 2]; w.w = o[ni][4 * a + 3];
                    po[(size_t)(ni * 8 + 2 * a + lh) * ROWS + row] = w;
                }
            if (lh == 0) {
                float* pm = part_ml + blk * (size_t)(2 * ROWS);
                pm[row] = m_run;
                pm[ROWS + row] = l_tot;
            }
        }
        return;
    }
    if (row_id < n_rows) {
        const float inv = 1.f / l_tot;
        bf16_t* op = out + (tok0 + tq) * q_stride + (size_t)(kvh * G + gq) * HD;
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                u32x2 w;
                w.x = pack_bf16x2(o[ni][4 * a] * inv, o[ni][4 * a + 1] * inv);
                w.y = pack_bf16x2(o[ni][4 * a + 2] * inv, o[ni][4 * a + 3] * inv);
                *reinterpret_cast<u32x2*>(op + ni * 32 + 8 * a + 4 * lh) = w;
            }
    }
    };   // unit

    if constexpr (!PERSIST) {
        unit(blockIdx.x, blockIdx.y, 0, 0, 0);
    } else {
        // consecutive shares (mostly the same kv head) on one XCD
        const int w = (blockIdx.x % 8) * (gridDim.x / 8) + blockIdx.x / 8;
        const int4 b = bounds[w], e = bounds[w + 1];
        const int n_items_all = tile_start[n_seq], n_items = n_items_all < max_items ? n_items_all : max_items;
        int kvh = b.x, item = b.y, t = b.z, slot = 2 * w;
        while (kvh < n_kv && (kvh != e.x || item != e.y || t < e.z)) {
            const bool last = kvh == e.x && item == e.y;
            unit(item, kvh, t, last ? e.z : INT_MAX, slot);
            if (last) break;
            t = 0;
            slot = 2 * w + 1;   // a share's first unit may be cut at its begin, its last at its end; none between
            if (++item >= n_items) item = 0, ++kvh;
        }
    }
}

// Merges the cut units of the persistent kernel: out = sum_p 2^(m_p - M) O_p / sum_p 2^(m_p - M) l_p over its parts p
// in key order, M = max_p m_p.  Workgroup (w, z) stands at the bound between shares w and w + 1; where that is the first
// cut of a unit it merges the unit's parts for HD / 4 columns, a thread per row.
template <int HD>
__global__ __launch_bounds__(LAPS_ATTN_LONG_ROWS) void attn_merge_cut_kernel(
    bf16_t* __restrict__ out, const float* __restrict__ part_o, const float* __restrict__ part_ml,
    const int4* __restrict__ desc, const int4* __restrict__ bounds, int n_wgs, int n_q, int n_kv, int n_tokens) {
    constexpr int ROWS = LAPS_ATTN_LONG_ROWS;
    constexpr int NC = HD / 16;   // 4-float chunks per thread
    const int w = blockIdx.x + 1;
    const int4 here = bounds[w];
    if (here.z == 0 || here.x >= n_kv) return;    // not inside a unit
    const int4 before = bounds[w - 1];
    const bool same = before.x == here.x && before.y == here.y;
    if (same && before.z > 0) return;             // the unit's first cut merges it
    const int4 it = desc[2 * here.y];
    const int G = n_q / n_kv, L = it.z, rs = desc[2 * here.y + 1].x;
    if (rs < 0 || L > n_tokens - rs) return;      // as in attn_kernel
    const int row = threadIdx.x, row_id = it.y * ROWS + row;
    if (row_id >= L * G) return;
    f32x4 acc[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_all = -INFINITY, l_all = 0.f;
    auto add = [&](int slot) {
        const float m = part_ml[(size_t)slot * 2 * ROWS + row], l = part_ml[(size_t)slot * 2 * ROWS + ROWS + row];
        const f32x4* po = reinterpret_cast<const f32x4*>(part_o) + ((size_t)slot * (HD / 4) + blockIdx.y * NC) * ROWS + row;
        f32x4 v[NC];
#pragma unroll
        for (int c = 0; c < NC; ++c) v[c] = po[(size_t)c * ROWS];
        const float m_new = fmaxf(m_all, m);
        const float a = __builtin_amdgcn_exp2f(m_all - m_new), b = __builtin_amdgcn_exp2f(m - m_new);
        l_all = l_all * a + l * b;
#pragma unroll
        for (int c = 0; c < NC; ++c) acc[c] = acc[c] * a + v[c] * b;
        m_all = m_new;
    };
    add(2 * (w - 1) + (same ? 0 : 1));            // the part before the cut: share w - 1's only unit, or its last one
    for (int v = w; v < n_wgs; ++v) {
        const int4 b = bounds[v], e = bounds[v + 1];
        if (b.x != here.x || b.y != here.y) break;
        if (e.x != b.x || e.y != b.y || e.z != b.z) add(2 * v);   // an empty share has written nothing
    }
    const float inv = 1.f / l_all;
    const int tq = row_id / G, gq = row_id - tq * G;
    bf16_t* op = out + ((size_t)rs + tq) * (size_t)(n_q * HD) + (size_t)(here.x * G + gq) * HD + blockIdx.y * NC * 4;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        u32x2 o2;
        o2.x = pack_bf16x2(acc[c].x * inv, acc[c].y * inv);
        o2.y = pack_bf16x2(acc[c].z * inv, acc[c].w * inv);
        *reinterpret_cast<u32x2*>(op + 4 * c) = o2;
    }
}

// Merges the key-range splits of attn_kernel<.., SPLIT = true> in a fixed order: out = sum_z 2^(m_z - M) O_z /
// sum_z 2^(m_z - M) l_z with M = max_z m_z.  A workgroup covers the 128 rows of one work item and CH 4-float
// slices of head_dim; its four groups of 128 threads take the splits z = g, g + 4, g + 8, ... (more loads in flight than one
// thread per row could issue) and their four partial sums are added in the order g = 0, 1, 2, 3.
constexpr int MERGE_GROUPS = 4;
constexpr int MERGE_SMALL = 512;   // workgroups
template <int HD, int CH>
__global__ __launch_bounds__(128 * MERGE_GROUPS) void attn_merge_kernel(
    bf16_t* __restrict__ out, const float* __restrict__ part_o, const float* __restrict__ part_ml,
    const int4* __restrict__ desc, int n_split, int n_q, int n_kv, int n_tokens) {
    constexpr int ROWS = 128;
    __shared__ float red_m[MERGE_GROUPS][ROWS];
    __shared__ float red_l[MERGE_GROUPS][ROWS];
    __shared__ f32x4 red_o[CH][MERGE_GROUPS][ROWS];
    const int item = blockIdx.x, kvh = blockIdx.y;
    const int4 it = desc[2 * item];
    const int4 at = desc[2 * item + 1];
    const int qtile = it.y, G = n_q / n_kv, L = it.z, rs = at.x, used = at.y;         // parts of the item
    if (it.x < 0 || rs < 0 || L > n_tokens - rs) return;                              // as in attn_kernel
    const int n_rows = L * G, R0 = qtile * ROWS;
    if (R0 >= n_rows) return;
    if (used == 1) return;   // the attention kernel wrote the final rows itself (uniform over the workgroup)
    const int row = threadIdx.x % ROWS, g = threadIdx.x / ROWS, row_id = R0 + row;
    const bool live = row_id < n_rows;
    const size_t blk0 = ((size_t)item * n_kv + kvh) * n_split;
    const float* pm = part_ml + blk0 * (size_t)(2 * ROWS) + row;
    // every load below is independent of the others: unrolled so that many are in flight at once
    float m_g = -INFINITY;
    if (live) {
#pragma unroll 4
        for (int z = g; z < used; z += MERGE_GROUPS) m_g = fmaxf(m_g, pm[(size_t)z * 2 * ROWS]);
    }
    red_m[g][row] = m_g;
    __syncthreads();
    float m_all = red_m[0][row];
#pragma unroll
    for (int k = 1; k < MERGE_GROUPS; ++k) m_all = fmaxf(m_all, red_m[k][row]);
    const int c0 = blockIdx.z * CH;
    const f32x4* po = reinterpret_cast<const f32x4*>(part_o) + (blk0 * (size_t)(HD / 4) + c0) * ROWS + row;
    f32x4 acc[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float l_g = 0.f;
    if (live) {
#pragma unroll 4
        for (int z = g; z < used; z += MERGE_GROUPS) {
            const float w = __builtin_amdgcn_exp2f(pm[(size_t)z * 2 * ROWS] - m_all);
            f32x4 v[CH];
#pragma unroll
            for (int c = 0; c < CH; ++c) v[c] = po[((size_t)z * (HD / 4) + c) * ROWS];
            l_g = __builtin_fmaf(w, pm[(size_t)z * 2 * ROWS + ROWS], l_g);
#pragma unroll
            for (int c = 0; c < CH; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[c][e] = __builtin_fmaf(w, v[c][e], acc[c][e]);
        }
    }
    red_l[g][row] = l_g;
#pragma unroll
    for (int c = 0; c < CH; ++c) red_o[c][g][row] = acc[c];
    __syncthreads();
    // group g finishes the slices g, g + 4, ...
    if (g >= CH || !live) return;
    float l_all = red_l[0][row];
#pragma unroll
    for (int k = 1; k < MERGE_GROUPS; ++k) l_all += red_l[k][row];
    const float inv = 1.f / l_all;
    const int tq = row_id / G, gq = row_id - tq * G;
    bf16_t* op = out + ((size_t)rs + tq) * (size_t)(n_q * HD) + (size_t)(kvh * G + gq) * HD;
    for (int c = g; c < CH; c += MERGE_GROUPS) {
        f32x4 o4 = red_o[c][0][row];
#pragma unroll
        for (int k = 1; k < MERGE_GROUPS; ++k) o4 += red_o[c][k][row];
        u32x2 o2;
        o2.x = pack_bf16x2(o4.x * inv, o4.y * inv);
        o2.y = pack_bf16x2(o4.z * inv, o4.w * inv);
        *reinterpret_cast<u32x2*>(op + 4 * (c0 + c)) = o2;
    }
}

template <int HD, int NW, bool HALVES = false>
int launch_attn(const bf16_t* q, bf16_t* out, const bf16_t* k_pool, const bf16_t* v_pool, const int4* desc,
                const int* page_table, int max_pages, const int* tile_start, int n_seq, int max_items, int n_q, int n_kv, int n_pool_pages, int n_tokens,
                hipStream_t s) {
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)HD);
    hipLaunchKernelGGL((attn_kernel<HD, NW, false, false, HALVES>), dim3(max_items, n_kv), dim3(NW * 64), 0, s, q, out, nullptr,
                       nullptr, k_pool, v_pool, desc, page_table, max_pages, tile_start,
                       n_seq, n_q, n_kv, scale_log2e, n_pool_pages, n_tokens, max_items, nullptr);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

template <int HD>
int launch_attn_persistent(const bf16_t* q, bf16_t* out, float* part, int n_wgs, const int4* bounds, const bf16_t* k_pool,
                           const bf16_t* v_pool, const int4* desc,
                           const int* page_table, int max_pages, const int* tile_start, int n_seq,
                           int max_items, int n_q, int n_kv, int n_pool_pages, int n_tokens, hipStream_t s) {
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)HD);
    float* part_ml = part + (size_t)2 * n_wgs * LAPS_ATTN_LONG_ROWS * HD;
    hipLaunchKernelGGL((attn_kernel<HD, 8, false, true>), dim3(n_wgs), dim3(512), 0, s, q, out, part, part_ml, k_pool, v_pool,
                       desc, page_table, max_pages, tile_start, n_seq, n_q, n_kv,
                       scale_log2e, n_pool_pages, n_tokens, max_items, bounds);
    LAPS_LAUNCH_CHECK();
    hipLaunchKernelGGL((attn_merge_cut_kernel<HD>), dim3(n_wgs - 1, 4), dim3(LAPS_ATTN_LONG_ROWS), 0, s, out, part, part_ml,
                       desc, bounds, n_wgs, n_q, n_kv, n_tokens);
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

template <int HD>
int launch_attn_split(const bf16_t* q, bf16_t* out, float* part, const bf16_t* k_pool, const bf16_t* v_pool,
                      const int4* desc, const int* page_table,
                      int max_pages, const int* tile_start, int n_seq, int max_items, int n_split,
                      int n_q, int n_kv, int n_pool_pages, int n_tokens, hipStream_t s) {
    const float scale_log2e = 1.4426950408889634f / sqrtf((float)HD);
    const size_t blocks = (size_t)max_items * n_kv * n_split;
    float* part_o = part;
    float* part_ml = part + blocks * 128 * HD;
    hipLaunchKernelGGL((attn_kernel<HD, 4, true, false>), dim3(max_items, n_kv, n_split), dim3(256), 0, s, q, out, part_o, part_ml,
                       k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq,
                       n_q, n_kv, scale_log2e, n_pool_pages, n_tokens, max_items, nullptr);
    LAPS_LAUNCH_CHECK();
    // slices of head_dim a workgroup merges: one where all of them are on the chip at once, four from there on
    if ((long)max_items * n_kv * (HD / 4) <= MERGE_SMALL) {
        hipLaunchKernelGGL((attn_merge_kernel<HD, 1>), dim3(max_items, n_kv, HD / 4), dim3(128 * MERGE_GROUPS), 0, s, out, part_o, part_ml,
                       desc, n_split, n_q, n_kv, n_tokens);
    } else {
        hipLaunchKernelGGL((attn_merge_kernel<HD, 4>), dim3(max_items, n_kv, HD / 16), dim3(128 * MERGE_GROUPS), 0, s, out, part_o, part_ml,
                       desc, n_split, n_q, n_kv, n_tokens);
    }
    LAPS_LAUNCH_CHECK();
    return LAPS_OK;
}

}  // namespace

// Upper bound on the workgroups of a key-split launch, and the bytes of partial results it needs.
static constexpr int kSplitTargetBlocks = 512;   // aim for two workgroups per compute unit
static constexpr int kSplitBelowBlocks = 256;    // launches with fewer un-split workgroups than this are split
static constexpr int kSplitMax = 64;

size_t laps_attn_partial_bytes(int hd, int max_pages) {
    // page tables too narrow for two splits never take the split path (same test as attn_blocking)
    if (((long)max_pages * LAPS_PAGE + KT - 1) / KT < 2 * MIN_TILES_PER_SPLIT) return 0;
    // blocks0 < kSplitBelowBlocks and n_split <= ceil(kSplitTargetBlocks / blocks0) give fewer than
    // kSplitTargetBlocks + kSplitBelowBlocks workgroups, each with 128 rows of (hd + 2) floats
    return (size_t)(kSplitTargetBlocks + kSplitBelowBlocks) * 128 * (size_t)(hd + 2) * sizeof(float);
}

// Query-row blocking for a batch: rows per workgroup (128 or 256), an upper bound on the number of
// (sequence, row block) work items, and the most parts an item's key range is split into.  Depends only on shapes known to
// the host (a captured graph must replay with the same grid whatever the lengths staged into it).
static void attn_blocking(int n_seq, int n_tokens, int group, int n_kv, int max_pages, int* mt, int* max_items,
                          int* n_split, int* min_tiles) {
    const long total_rows = (long)n_tokens * group;
    const long items1 = total_rows / 128 + n_seq;      // bound with 128-row blocks
    const int max_kv_tiles = (max_pages * LAPS_PAGE + KT - 1) / KT;
    *n_split = 1;
    *min_tiles = MIN_TILES_PER_SPLIT;
    if (items1 * n_kv < kSplitBelowBlocks && max_kv_tiles >= 2 * MIN_TILES_PER_SPLIT) {
        const int blocks0 = (int)items1 * n_kv;
        // A turn or two of few tokens leave most compute units idle however fine the split: a workgroup per key tile where all
        // of them fit one round, as wide as the page table is, and the rows of their partial results are few.  Attention with
        // its scheduling kernel, splits of at least 4 tiles and of one: 7B, a turn of 7 over 900 / 2000 / 4000 keys 17.5 / 16.7 /
        // 18.4 and 13.2 / 13.4 / 16.7; 14B, 7 rows over 900 keys with the rest of its one-layer graph 148.3 and 143.6 (a table of
        // 129 pages and more leaves that at 4 tiles).  Not for more workgroups (32B, 2 turns of 32 over 2000 keys 26.3 / 28.2) or
        // rows (7B, a turn of 16 over 4000 keys, 64 x 112 rows, 19.5 / 20.4; tiny model, 64 x 128, 14.5 / 14.8; 48 x 128 still
        // 15.2 / 13.8).
        if ((long)blocks0 * max_kv_tiles <= 256 && total_rows * max_kv_tiles <= 6400) *min_tiles = 1;
        int ns = (kSplitTargetBlocks + blocks0 - 1) / blocks0;
        ns = ns < max_kv_tiles / *min_tiles ? ns : max_kv_tiles / *min_tiles;
        ns = ns < kSplitMax ? ns : kSplitMax;
        if (ns > 1) {
            *n_split = ns;
            *mt = 1;
            *max_items = (int)items1;
            return;
        }
    }
    // Few key tiles: 256-row blocks pay for their pipelined loop (three stages to fill and drain) and for the rows that fill
    // no block; 128-row blocks pay by reading the keys twice and without the pipeline.  Up to the split's 8 tiles 128 rows are
    // the faster ones where each block has a compute unit (256- against 128-row blocks, attention with its scheduling kernel:
    // 32B, 8 turns of 64 in 440 keys 29.2 and 24.3 us, a prompt of 440 27.5 and 23.6).  With more blocks than units 5 to 7 tiles
    // are the pipeline's (12 turns of 100 in 440 keys 31.5 and 35.0).  Up to 4 tiles 128 rows win where they spare a quarter of
    // the rows (40 turns of 64 in 256 keys 40.5 and 31.5) or take more than one round of two blocks a unit: ragged turns by
    // 1.08 to 1.25 (47 turns of 33 to 64 over up to 100 keys 42.3 and 33.8); lost are batches of equal lengths that fill rounds
    // of 256-row blocks exactly (7B, 64 turns of 64 in 256 keys 49.7 and 52.0).  Between, ragged batches gain or lose 3 %, equal
    // ones lose up to 10 %.  Up to 2 tiles 128 rows always win (64 prompts of 64 tokens 44.0 and 37.4).
    const long blocks1 = items1 * n_kv;
    const bool spares = total_rows > 256L * n_seq && total_rows <= 384L * n_seq;   // 3 blocks of 128 rows instead of 2 of 256
    const bool few = max_kv_tiles <= 2 || (max_kv_tiles <= 4 && (spares || blocks1 > 512)) ||
                     (max_kv_tiles < 2 * MIN_TILES_PER_SPLIT && blocks1 <= 256);
    *mt = (!few && total_rows > 128L * n_seq) ? 2 : 1;  // average rows per sequence above one 128-row block
    const int rows_per_wg = 128 * *mt;
    // every sequence contributes ceil(rows/rows_per_wg) blocks: at most rows/rows_per_wg + 1
    *max_items = (int)(total_rows / rows_per_wg) + n_seq;
}

void laps_attn_plan(int n_seq, int n_tokens, int group, int n_kv, int max_pages, int* rows_per_wg, int* max_items,
                    int* n_split, int* min_tiles_per_split) {
    int mt = 1;
    attn_blocking(n_seq, n_tokens, group, n_kv, max_pages, &mt, max_items, n_split, min_tiles_per_split);
    *rows_per_wg = 128 * mt;
}

// Work-item table for laps_launch_attention; depends on the batch only, so a layer stack builds it once.
static size_t item_table_ints(int max_tokens, int max_seqs, int group) {   // items of the smallest blocking, 16-byte units
    return (((size_t)max_tokens * group / 128 + max_seqs + 2) + 3) / 4 * 4;
}
size_t laps_attn_item_table_bytes(int max_tokens, int max_seqs, int group) {
    const size_t n = item_table_ints(max_tokens, max_seqs, group);
    return 2 * n * sizeof(int) + (LAPS_ATTN_MAX_WGS + 1 + 2 * n) * sizeof(int4);
}
void laps_attn_item_tables(int* item_seq, int n_tokens, int n_seq, int group, int** pre, int4** bounds, int4** desc) {
    const size_t n = item_table_ints(n_tokens, n_seq, group);
    *pre = item_seq + n;
    *bounds = reinterpret_cast<int4*>(item_seq + 2 * n);
    *desc = *bounds + LAPS_ATTN_MAX_WGS + 1;
}

// The persistent kernel takes un-split launches of 256-row blocks where units differ enough in length for equal shares to
// outweigh the merge launch and the cuts: with a grid of units, the last partly filled round of workgroups and the longest
// units leave compute units idle.  32B shape (head_dim 128, 40 / 8 heads), attention alone with its scheduling kernels,
// grid of units against equal shares: 2048 rows over 2048 keys 223 -> 174 us, 1847 rows over 6144 444 -> 308, 12 short
// turns (573 rows) over up to 4096 keys 130 -> 71, 64 turns 334 -> 297, 2048 rows without a prefix 106 -> 94.
// MIN_TILES_PERSIST: with tables of 16 tiles (prefixes of up to 960 keys) 16 / 40 / 64 turns of the 32B shape take 49 / 61 /
// 83 us in shares and 44 / 67 / 93 on the grid, 30 longer turns of the 7B shape 80 and 74; with 24 tiles 56 / 78 / 106 and
// 58 / 92 / 120, 92 and 102.
// One sequence whose units have a workgroup each stays with the grid where its shares would not be cut with the longest
// prefix the page table holds (with a shorter one even less): 1000 rows without a prefix 57 us in cut shares, 46 on the
// grid; 1500 over 2048 keys 135 and 123.
constexpr int MIN_TILES_PERSIST = 20;
constexpr int GRID_CUT_COST = 20;   // what cutting costs against the grid: the merge launch comes on top
int laps_attn_persistent_wgs(int n_seq, int n_tokens, int group, int n_kv, int hd, int max_pages, size_t partial_bytes) {
    int mt, max_items, n_split, min_tiles;
    attn_blocking(n_seq, n_tokens, group, n_kv, max_pages, &mt, &max_items, &n_split, &min_tiles);
    const long tiles = (max_pages * (long)LAPS_PAGE + KT - 1) / KT;
    if (mt != 2 || n_split != 1 || tiles < MIN_TILES_PERSIST) return 0;
    const size_t slot = (size_t)LAPS_ATTN_LONG_ROWS * (hd + 2) * sizeof(float);
    size_t room = partial_bytes / (2 * slot) / 8 * 8;   // whole groups of the 8 XCDs; 192 at least in a workspace for these tables
    const int wgs = room < LAPS_ATTN_MAX_WGS ? (int)room : LAPS_ATTN_MAX_WGS;
    const int items = (n_tokens * group + LAPS_ATTN_LONG_ROWS - 1) / LAPS_ATTN_LONG_ROWS;
    if (n_seq == 1 && items * n_kv <= wgs) {
        const long room_h = max_pages * (long)LAPS_PAGE - n_tokens, h = room_h > 0 ? room_h : 0;
        long cost = 0, longest = 0;
        for (int i = 1; i <= items; ++i) {
            const int rows = i * LAPS_ATTN_LONG_ROWS < n_tokens * group ? i * LAPS_ATTN_LONG_ROWS : n_tokens * group;
            longest = (h + (rows - 1) / group + KT) / KT + LAPS_ATTN_COST0;
            cost += longest * n_kv;
        }
        if (longest <= cost / wgs + GRID_CUT_COST) return 0;
    }
    return wgs;
}

int laps_launch_attention(const bf16_t* q, bf16_t* out, const bf16_t* k_pool, const bf16_t* v_pool,
                          const int* page_table, int max_pages, int n_seq, int n_tokens, const int* tile_start,
                          const int* item_seq, float* partial, size_t partial_bytes, int n_q, int n_kv, int hd, int n_pool_pages,
                          hipStream_t s) {
    int mt, max_items, n_split, min_tiles;
    attn_blocking(n_seq, n_tokens, n_q / n_kv, n_kv, max_pages, &mt, &max_items, &n_split, &min_tiles);
    const int n_wgs = partial ? laps_attn_persistent_wgs(n_seq, n_tokens, n_q / n_kv, n_kv, hd, max_pages, partial_bytes) : 0;
    int* pre;
    int4 *bounds, *desc;
    laps_attn_item_tables(const_cast<int*>(item_seq), n_tokens, n_seq, n_q / n_kv, &pre, &bounds, &desc);
    if (n_wgs > 0) {
        auto launch = hd == 128 ? launch_attn_persistent<128> : launch_attn_persistent<64>;
        return launch(q, out, partial, n_wgs, bounds, k_pool, v_pool, desc, page_table, max_pages,
                      tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
    }
    if (n_split > 1) {
        if (!partial) {
            laps_set_error("attention: key-split launch needs the partial-result workspace");
            return LAPS_EINVAL;
        }
        if (hd == 128) return launch_attn_split<128>(q, out, partial, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_split, n_q, n_kv, n_pool_pages, n_tokens, s);
        if (hd == 64) return launch_attn_split<64>(q, out, partial, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_split, n_q, n_kv, n_pool_pages, n_tokens, s);
    }
    // 128-row blocks that would be 256-row ones over more key tiles: summed up as those do, so that the width of the page table
    // does not show in the result (the sums of rounded probabilities are also the ones that match the second product:
    // 32B prompts of 64 tokens 1.79e-3 from 64 bits, with sums of unrounded ones 1.81e-3; the same time)
    const bool halves = (long)n_tokens * (n_q / n_kv) > 128L * n_seq;
    if (hd == 128) {
        if (mt == 2) return launch_attn<128, 8>(q, out, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
        if (halves) return launch_attn<128, 4, true>(q, out, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
        return launch_attn<128, 4>(q, out, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
    }
    if (hd == 64) {
        if (mt == 2) return launch_attn<64, 8>(q, out, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
        if (halves) return launch_attn<64, 4, true>(q, out, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
        return launch_attn<64, 4>(q, out, k_pool, v_pool, desc, page_table, max_pages, tile_start, n_seq, max_items, n_q, n_kv, n_pool_pages, n_tokens, s);
    }
    laps_set_error("attention: head_dim %d not supported (64 or 128)", hd);
    return LAPS_EINVAL;
}
