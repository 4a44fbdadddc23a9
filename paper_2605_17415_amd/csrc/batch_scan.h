// The kernel of the query-batched list scan, one instantiation per (panel width, stored bits); included by the
// translation units batch_scan_b*.hip, which compile the widths of one bit count each.
//
// One workgroup takes one list and up to TQ of the queries that probe it: the de-quantised codes of 32 or 64
// vectors are one MFMA operand (held in registers and reused for every query tile), the rotated queries are the
// other (a panel in LDS).
//
// Arithmetic: both operands are used in split float16 form, 1024*v = hi + lo with hi = fp16(1024 v)
// and lo = fp16(1024 v - hi), and the product is accumulated as hi*hi + hi*lo + lo*hi on
// v_mfma_f32_32x32x16_f16 with float32 accumulation (the lo*lo term, below 2^-24 relative, is
// dropped).  Each part carries 11 significant bits, so the result matches a float32 contraction to
// about 2e-7 relative while running on the float16 matrix pipe; the 2^-20 of the two scale factors
// is folded into the stored norm.
//
// v_mfma_f32_32x32x16_f16: A is 32x16 (lane = i + 32*(k/8), element k%8), B is 16x32 likewise,
// D as for the 32x32 float32 form: D[i][j] in lane j + 32*((i/4)%2), register (i%4) + 4*(i/8).
#pragma once
#include <hip/hip_fp16.h>

#include <type_traits>

#include "kernels.h"

namespace ivftq {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

namespace {

// Copies of the table of code pairs in a threshold pass that is worth them (run_batch).  Entry e's c-th lies at e * copies + c and a
// lane reads copy lane % copies, so that the 64 lanes of a look-up, each with a pair of its own, collide on fewer banks.
// Clocks of a compute unit per look-up by two workgroups, 256 entries: 1 copy 7.5, 2 8.1, 4 6.6, 8 6.0, 16 4.4, 32 4.4.
constexpr int kTableCopies = 16;
constexpr int64_t kCopiesFrom = 400'000'000;       // coordinates de-quantised by a pass from which their making is paid back

template <int DP, int B, int NQ>
struct BatchCfg {
    static constexpr int TQ = NQ * 32;
    static constexpr int LDH = DP + 8;            // halves per panel row: 16-byte pad keeps b128 reads conflict free
    static constexpr bool PAIR = B <= 5;          // two codes per table look-up
    static constexpr int PT = PAIR ? 1 << (2 * B) : 1 << B;
    // dense pass: both parts of the panel, and table entries of both parts (two codes: 8 bytes, one code: 4)
    static constexpr size_t lds_dense = (size_t)2 * TQ * LDH * sizeof(uint16_t) + 16 * TQ + (size_t)PT * (PAIR ? 8 : 4);
    // LDS of a workgroup when a compute unit holds `occ` of them (in whole allocation units, less the passes' static words)
    static constexpr size_t room(int occ) { return 160 * 1024 / occ / 1280 * 1280 - 64; }
    // Threshold pass: hi parts of the panel, the table, perhaps in several copies, and (hold) candidates of a tile held back in
    // what is left of the room, at most 4096.
    static constexpr size_t panel_threshold = (size_t)TQ * LDH * sizeof(uint16_t) + 16 * TQ, table_threshold = (size_t)PT * 4;
    static constexpr int held_back(int occ, int copies) {
        const size_t fit = (room(occ) - panel_threshold - copies * table_threshold - 4 * TQ) / 8;
        return fit < 4096 ? (int)fit / 2 * 2 : 4096;
    }
    static constexpr size_t lds_threshold(int occ, bool hold, int copies) {
        return panel_threshold + copies * table_threshold + (hold ? 8 * (size_t)held_back(occ, copies) + 4 * TQ : 0);
    }
    static constexpr bool copies_fit(int occ, bool hold) { return lds_threshold(occ, false, kTableCopies) + (hold ? 8 * 400 + 4 * TQ : 0) <= room(occ); }
};

// The 8 codes of block kb that a lane de-quantises, coordinates 16*kb + 8*half + [0, 8), begin in word first_word
// at bit first_bit.
template <int B> __host__ __device__ constexpr int first_word(int kb, int half) { return ((16 * kb + 8 * half) * B) >> 5; }
template <int B> __host__ __device__ constexpr int first_bit(int kb, int half) { return ((16 * kb + 8 * half) * B) & 31; }

template <int B, int NW>
__device__ __forceinline__ uint64_t code_chunk(const uint32_t (&w)[NW], int kb, int half) {
    const int sh = half ? first_bit<B>(kb, 1) : first_bit<B>(kb, 0);
    if constexpr (NW == 1) return w[0] >> sh;      // B = 2 or 4: the codes end inside the word
    else return (((uint64_t)w[1] << 32) | w[0]) >> sh;
}

// Which part of which list, and which queries, one tile of a pass covers.
struct BatchTile {
    int l, v_lo, v_hi, nq_tile;          // vectors [v_lo, v_hi) of list l; v_lo is a multiple of 64
    int64_t pair0, base_slot;
    __device__ __forceinline__ void find(const BatchScanArgs& a, int tile, int tq) {
        const int bkt = (a.dense ? a.p.tile_near : a.p.tile_late)[tile];
        l = bkt >= a.L ? bkt - a.L : bkt;
        const int n_l = a.store.list_size[l], parts = list_parts(n_l, a.part_len), rel = tile - a.p.tile_off[bkt];
        const int len = ((n_l + parts - 1) / parts + 63) & ~63;
        v_lo = (rel % parts) * len;
        v_hi = v_lo + len < n_l ? v_lo + len : n_l;
        const int skip = rel / parts * tq, left = (int)a.p.count[bkt] - skip;
        pair0 = (int64_t)a.p.pair_off[bkt] + skip;
        nq_tile = left < tq ? left : tq;
        base_slot = a.store.list_off[l];
    }
};

// The workgroups of a launch are as many as the chip holds and take tiles from a common counter until none is
// left: tiles differ in work by the sizes of the lists and the queries that meet there, and with a workgroup per
// tile the compute units stood idle for 22 % of the passes at 10M x 96 (waiting for the last ones), the launch
// besides being sized for the most tiles there could be.  The next number is fetched while a tile is worked on.
struct TileQueue {
    const BatchScanArgs& a;
    int* s_next;                         // [2] in LDS
    int turn = 0, end;
    __device__ __forceinline__ TileQueue(const BatchScanArgs& args, int* lds) : a(args), s_next(lds) {
        end = a.p.totals[a.dense ? 1 : 2];
        request();
    }
    __device__ __forceinline__ void request() {
        if (threadIdx.x == 0) s_next[turn] = atomicAdd(&a.p.totals[a.dense ? 3 : 4], 1);
    }
    // the tile to work on (past `end`: none); a barrier for the workgroup
    __device__ __forceinline__ int take() {
        __syncthreads();
        const int tile = s_next[turn];
        turn ^= 1;
        return __builtin_amdgcn_readfirstlane(tile);
    }
};

// Queries of the tile: word e of s_row as given by `word` for pair number `it` (or `none` beyond the tile), then
// the rotated coordinates (zero beyond the tile and beyond the padded width of the query rows).
template <int DP, int TQ, int NT, bool LO, class Word>
__device__ __forceinline__ void stage_queries(const BatchScanArgs& a, const BatchTile& t, uint16_t* zh, uint16_t* zl, uint4* s_row,
                                              uint4 none, Word word) {
    constexpr int LDH = DP + 8;
    int tid = threadIdx.x;
    asm volatile("" : "+v"(tid));        // or what follows from it is computed once and kept in registers from tile to tile
    for (int e = tid; e < TQ; e += NT) s_row[e] = e < t.nq_tile ? word(a.p.pairs[t.pair0 + e]) : none;
    for (int e = tid; e < TQ * (DP / 8); e += NT) {           // 16-byte pieces
        const int r = e / (DP / 8), c8 = e % (DP / 8);
        uint4 vh = make_uint4(0, 0, 0, 0), vl = make_uint4(0, 0, 0, 0);
        if (r < t.nq_tile && c8 * 8 < a.z_pitch) {
            const int64_t at = (int64_t)(a.p.pairs[t.pair0 + r] / a.np) * a.z_pitch + c8 * 8;
            vh = *reinterpret_cast<const uint4*>(a.zh + at);
            if (LO) vl = *reinterpret_cast<const uint4*>(a.zl + at);
        }
        *reinterpret_cast<uint4*>(zh + r * LDH + c8 * 8) = vh;
        if (LO) *reinterpret_cast<uint4*>(zl + r * LDH + c8 * 8) = vl;
    }
}

// Words of a slab of 32 vectors (slots first_slot ... + 31) as lane jl of either half de-quantises them.  Blocks
// whose words exist for both halves of the wavefront (the same for every lane) are loaded at constant offsets with
// no tests in between: all of them when the rows are as long as the panel, all but the last for a row that ends
// inside the last block (d = 200 in a 208-wide panel); else block by block.
// (The upper half's words lie a fixed 0, 1 or 2 words after the lower half's, so a lane needs one pointer per such
// distance and every load has a constant offset.)
template <int KB, int B, int NW>
__device__ __forceinline__ void fetch_words(const uint32_t* wp, int words, int half, uint32_t (&w)[KB][NW]) {
    const uint32_t* const up[3] = {wp, wp + 64 * half, wp + 128 * half};
    auto whole = [&](int kb) { return first_word<B>(kb, 1) + NW - 1 < words; };
    auto block = [&](int kb) {
        const uint32_t* p = up[first_word<B>(kb, 1) - first_word<B>(kb, 0)] + first_word<B>(kb, 0) * 64;
#pragma unroll
        for (int e = 0; e < NW; ++e) w[kb][e] = p[e * 64];
    };
    auto tested = [&](int kb) {
        const uint32_t* p = up[first_word<B>(kb, 1) - first_word<B>(kb, 0)] + first_word<B>(kb, 0) * 64;
        const int wi = half ? first_word<B>(kb, 1) : first_word<B>(kb, 0);
#pragma unroll
        for (int e = 0; e < NW; ++e) w[kb][e] = wi + e < words ? p[e * 64] : 0u;
    };
    if (whole(KB - 1)) {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) block(kb);
    } else if (KB > 1 && whole(KB - 2)) {
#pragma unroll
        for (int kb = 0; kb < KB - 1; ++kb) block(kb);
        tested(KB - 1);
    } else {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            if (whole(kb)) block(kb); else tested(kb);
        }
    }
}

// ---- dense pass: every score of the nearest lists is stored -------------------------------------------
//
// A list is among the nearest of few queries (three at 10M x 96 with 10,000 queries), so what bounds the pass is
// de-quantising: one LDS look-up per code pair whose 64 lanes collide on the banks (counters at 10M x 96 with
// separate tables for the two parts: LDS busy 63 % of the cycles, over half of that conflicts, matrix pipe 23 %).
// Both parts of a pair therefore sit in one 8-byte entry.  The queries are the row operand and the vectors the
// column operand, so a lane holds one vector's scores against 16 queries and the stores of a query's scores
// coalesce.
template <int DP, int B, int NQ, int WAVES, int OCC>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_batch_dense(BatchScanArgs a) {
    using Cfg = BatchCfg<DP, B, NQ>;
    constexpr int KB = DP / 16, NT = WAVES * 64;
    constexpr int NW = (B == 2 || B == 4) ? 1 : 2;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint16_t* zh = reinterpret_cast<uint16_t*>(lds_raw);                       // [TQ][LDH] hi parts of the rotated queries
    uint16_t* zl = zh + Cfg::TQ * Cfg::LDH;                                      // [TQ][LDH] lo parts
    uint4* s_row = reinterpret_cast<uint4*>(zl + Cfg::TQ * Cfg::LDH);          // [TQ] coarse term, first score's place (2 words), |q|
    uint2* tab = reinterpret_cast<uint2*>(s_row + Cfg::TQ);                      // [PT] (hi pair, lo pair); one code: [PT] words hi | lo << 16

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, half = lane >> 5, jl = lane & 31;
    constexpr float kUnscale = 1.f / (kSplitScale * kSplitScale);

    for (int e = tid; e < Cfg::PT; e += NT) {
        uint32_t hp = 0, lp = 0;
#pragma unroll
        for (int i = 0; i < (Cfg::PAIR ? 2 : 1); ++i) {
            const float V = a.cb[(e >> (i * B)) & ((1 << B) - 1)] * kSplitScale;
            const _Float16 hi = (_Float16)V;
            const _Float16 lo = (_Float16)(V - (float)hi);
            hp |= (uint32_t)__builtin_bit_cast(uint16_t, hi) << (16 * i);
            lp |= (uint32_t)__builtin_bit_cast(uint16_t, lo) << (16 * i);
        }
        if (Cfg::PAIR) tab[e] = make_uint2(hp, lp);
        else reinterpret_cast<uint32_t*>(tab)[e] = hp | (lp << 16);
    }
    const uint16_t* bh_base = zh + jl * Cfg::LDH + 8 * half;
    const uint16_t* bl_base = zl + jl * Cfg::LDH + 8 * half;
    __shared__ __align__(16) int s_next[4];      // (16 bytes: the panel behind it keeps its alignment)
    TileQueue queue(a, s_next);
    for (int tile; (tile = queue.take()) < queue.end;) {
    BatchTile t;
    t.find(a, tile, Cfg::TQ);
    const int v_lo = t.v_lo, v_hi = t.v_hi, nslab = (v_hi - v_lo + 31) / 32, n_qt = (t.nq_tile + 31) / 32;

    // Raw words and norm of a slab are fetched one slab ahead, so that their latency hides behind the current one.
    auto fetch = [&](int slab, uint32_t (&w)[KB][NW], uint32_t& g) {
        const int v = v_lo + slab * 32 + jl;
        const int64_t slot = t.base_slot + (v < v_hi ? v : v_hi - 1);
        fetch_words<KB, B, NW>(a.store.codes + (slot >> 6) * a.store.words * 64 + (slot & 63), a.store.words, half, w);
        g = a.store.gamma[slot];
    };
    uint32_t cw[KB][NW], nw[KB][NW], cg, ng;
    int slab = wave;
    if (slab < nslab) fetch(slab, cw, cg);

    stage_queries<DP, Cfg::TQ, NT, true>(a, t, zh, zl, s_row, make_uint4(0, 0, 0, 0), [&](int32_t it) {
        const int32_t q = it / a.np;
        const int64_t at = (int64_t)q * a.m_stride + a.cand_off[(int64_t)q * (a.np + 1) + (it - q * a.np)];
        return make_uint4(__float_as_uint(a.coarse[it]), (uint32_t)at, (uint32_t)(at >> 32), a.metric ? __float_as_uint(a.qnorm[q]) : 0u);
    });
    __syncthreads();
    queue.request();

    while (slab < nslab) {
        const int next = slab + WAVES;
        if (next < nslab) fetch(next, nw, ng);
        half8 ah[KB], al[KB];
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            const uint64_t chunk = code_chunk<B, NW>(cw[kb], kb, half);
            uint32_t hv[4], lv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                if constexpr (Cfg::PAIR) {
                    const uint2 e = tab[(uint32_t)(chunk >> (2 * B * i)) & (uint32_t)(Cfg::PT - 1)];
                    hv[i] = e.x;
                    lv[i] = e.y;
                } else {
                    const uint32_t* one = reinterpret_cast<const uint32_t*>(tab);
                    const uint32_t e0 = one[(uint32_t)(chunk >> (2 * B * i)) & (uint32_t)(Cfg::PT - 1)];
                    const uint32_t e1 = one[(uint32_t)(chunk >> (2 * B * i + B)) & (uint32_t)(Cfg::PT - 1)];
                    hv[i] = __builtin_amdgcn_perm(e1, e0, 0x05040100u);
                    lv[i] = __builtin_amdgcn_perm(e1, e0, 0x07060302u);
                }
            }
            ah[kb] = __builtin_bit_cast(half8, make_uint4(hv[0], hv[1], hv[2], hv[3]));
            al[kb] = __builtin_bit_cast(half8, make_uint4(lv[0], lv[1], lv[2], lv[3]));
        }
        const float g = kUnscale * __half2float(__ushort_as_half((uint16_t)cg));      // 2^-20 * norm of this lane's vector
        const int v = v_lo + slab * 32 + jl;
        float xn = 0.f;
        if (a.metric) xn = a.store.xnorm[t.base_slot + (v < v_hi ? v : v_hi - 1)];
        for (int qt = 0; qt < n_qt; ++qt) {
            floatx16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.f;
            const uint16_t* bhq = bh_base + qt * 32 * Cfg::LDH;
            const uint16_t* blq = bl_base + qt * 32 * Cfg::LDH;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const half8 bh = *reinterpret_cast<const half8*>(bhq + 16 * kb);
                const half8 bl = *reinterpret_cast<const half8*>(blq + 16 * kb);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, ah[kb], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(bl, ah[kb], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(bh, al[kb], acc, 0, 0, 0);
            }
            // (panel reads two blocks ahead of the products, see the threshold pass)
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            }
            // result row r of this lane: query 8*(r/4) + 4*half + r%4 of the tile, vector jl of the slab
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                // rows 4g .. 4g+3 belong to the queries 8g .. 8g+7 of this tile: a sparse tile (a list that
                // is among the nearest of few queries) skips the groups it has no query for
                if (qt * 32 + 8 * (r / 4) >= t.nq_tile) break;
                const int e = qt * 32 + 8 * (r / 4) + 4 * half + (r % 4);
                const uint4 row = s_row[e];
                float sc = fmaf(g, acc[r], __uint_as_float(row.x));
                if (a.metric) sc = metric_key(a.metric, sc, xn, __uint_as_float(row.w));
                if (e < t.nq_tile && v < v_hi) a.scores[(int64_t)(((uint64_t)row.z << 32) | row.y) + v] = sc;
            }
        }
#pragma unroll
        for (int kb = 0; kb < KB; ++kb)
#pragma unroll
            for (int e = 0; e < NW; ++e) cw[kb][e] = nw[kb][e];
        cg = ng;
        slab = next;
    }
    }
}

// ---- threshold pass: the other lists, only scores that can reach the query's threshold kept ------------
//
// The vectors are the row operand, so a lane holds one query's scores against 16 vectors and needs that query's
// coarse term and threshold only once.  Only the leading float16 parts are multiplied (one product instead of
// three): acc0 = 2^20 * kappa is added to the accumulators, kappa bounding the error of such a sum for a unit query,
// so what is compared with the threshold and appended is an upper bound of the true score (true score in
// [u - 2*kappa*gamma, u]); k_merge re-scores from the packed codes the few that can still matter.
//
// A wavefront takes a storage block of 64 vectors at a time, two row tiles (S = 2), so that every panel row it reads
// from LDS feeds two matrix instructions: with one row tile a panel read (8 LDS cycles, shared by four SIMDs) per
// matrix instruction (32 cycles) alone would keep LDS as busy as the matrix pipes, and the look-ups come on top.
// S = row tiles per wavefront (one where the registers do not reach for two).  RAW: scores are ranking keys of a raw
// metric (a template parameter: the lengths' range takes registers).
//
// A candidate is appended to its query's list with an update of the query's counter.  Updates of one counter from all over
// the chip follow each other at about 0.2 us, which is what the pass takes where candidates are many and queries
// few.  HOLD keeps the candidates of a tile in LDS and updates a counter once per tile (rows without clusters, 1M x
// 128, inner product, 100 queries of 64 probes, k = 100, up to 1172 candidates a query: 203 -> 104 us); what does not fit is
// appended at once.  It is left out where its registers would spill (the 96-wide panel at three wavefronts per SIMD).
// TC: copies of the table.
template <int DP, int B, int NQ, int WAVES, int OCC, int S, bool RAW, bool HOLD, int TC>
__global__ __launch_bounds__(WAVES * 64) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_batch_threshold(BatchScanArgs a) {
    using Cfg = BatchCfg<DP, B, NQ>;
    constexpr int KB = DP / 16, NT = WAVES * 64, VB = 32 * S;      // vectors of a block
    constexpr int CAND = Cfg::held_back(OCC, TC);
    constexpr int NW = (B == 2 || B == 4) ? 1 : 2;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint16_t* zh = reinterpret_cast<uint16_t*>(lds_raw);                       // [TQ][LDH] hi parts of the rotated queries
    uint4* s_row = reinterpret_cast<uint4*>(zh + Cfg::TQ * Cfg::LDH);          // [TQ] coarse term, threshold, pair number, |q|
    uint32_t* tab = reinterpret_cast<uint32_t*>(s_row + Cfg::TQ);                // [PT][TC] hi parts of a code pair, packed (or of one code)
    uint2* s_cand = reinterpret_cast<uint2*>(tab + Cfg::PT * TC);                     // HOLD: [CAND] score bits; column | vector of the part << 7 | place among the column's << 19
    int* s_cnt = reinterpret_cast<int*>(s_cand + CAND);                          // HOLD: [TQ] held back per column, then their first position
    static_assert(Cfg::TQ <= 128 && kPartMax <= 4096, "fields of a candidate held back");

    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, half = lane >> 5, jl = lane & 31;
    constexpr float kUnscale = 1.f / (kSplitScale * kSplitScale);

    for (int e = tid; e < Cfg::PT * TC; e += NT) {
        uint32_t hp = 0;
#pragma unroll
        for (int i = 0; i < (Cfg::PAIR ? 2 : 1); ++i)
            hp |= (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)(a.cb[(e / TC >> (i * B)) & ((1 << B) - 1)] * kSplitScale)) << (16 * i);
        tab[e] = hp;
    }
    const uint16_t* bh_base = zh + jl * Cfg::LDH + 8 * half;
    const uint32_t* mine = tab + tid % TC;
    const int words = a.store.words;
    __shared__ __align__(16) int s_next[4];      // (16 bytes: the panel behind it keeps its alignment) [2] asked for, [3] held back if that is too many
    TileQueue queue(a, s_next);
    if (HOLD && tid < Cfg::TQ) s_cnt[tid] = 0;
    if (HOLD && tid == 0) { s_next[2] = 0; s_next[3] = CAND; }
    BatchTile t{};
    for (;;) {
    const int tile = queue.take();
    if (HOLD && s_next[2] > 0) {                 // what the tile before held back, whose queries are still there
        const int held = s_next[2] <= CAND ? s_next[2] : s_next[3];      // (once one did not fit, none after it did)
        int me = threadIdx.x;
        asm volatile("" : "+v"(me));             // or what follows from it is computed ahead of the tiles and kept
        if (me < Cfg::TQ && s_cnt[me] > 0) s_cnt[me] = atomicAdd(&a.cand_cnt[(int32_t)s_row[me].z / a.np], s_cnt[me]);
        __syncthreads();
        for (int i = me; i < held; i += NT) {
            const uint2 c = s_cand[i];
            const int e = (int)(c.y & 127u);
            const int32_t it = (int32_t)s_row[e].z, q = it / a.np;
            const int pos = s_cnt[e] + (int)(c.y >> 19);
            if (pos < a.cap) {
                a.cand_score[(int64_t)q * a.cap + pos] = __uint_as_float(c.x);
                a.cand_slot[(int64_t)q * a.cap + pos] = (t.base_slot + t.v_lo + (int)((c.y >> 7) & 4095u)) | (int64_t)(it - q * a.np) << kCandProbeShift;
            }
        }
        __syncthreads();
        if (me < Cfg::TQ) s_cnt[me] = 0;
        if (me == 0) { s_next[2] = 0; s_next[3] = CAND; }
    }
    if (tile >= queue.end) break;
    t.find(a, tile, Cfg::TQ);
    const int v_lo = t.v_lo, v_hi = t.v_hi, nblk = (v_hi - v_lo + VB - 1) / VB, n_qt = (t.nq_tile + 31) / 32;

    // A list starts at a multiple of 64 slots and its slots reach to one, so a block's words and norms can be read
    // whole; what lies beyond the list is replaced by NaN norms below.
    const uint32_t* codes = a.store.codes + ((t.base_slot + v_lo) >> 6) * words * 64 + jl;
    uint32_t cw[S][KB][NW];
    int blk = wave;
    auto fetch = [&](int b) {
        const uint32_t* at = codes + (int64_t)((b * VB) >> 6) * words * 64 + ((b * VB) & 63);
#pragma unroll
        for (int s = 0; s < S; ++s) fetch_words<KB, B, NW>(at + 32 * s, words, half, cw[s]);
    };
    if (blk < nblk) fetch(blk);
    // (columns beyond the tile's queries: a NaN threshold, which not even an infinite score reaches)
    stage_queries<DP, Cfg::TQ, NT, false>(a, t, zh, nullptr, s_row, make_uint4(0, 0x7FC00000u, 0, 0), [&](int32_t it) {
        const int32_t q = it / a.np;
        return make_uint4(__float_as_uint(a.coarse[it]), __float_as_uint(a.thresh[(int64_t)q * a.thresh_stride]), (uint32_t)it,
                          RAW ? __float_as_uint(a.qnorm[q]) : 0u);
    });
    __syncthreads();
    queue.request();

    constexpr int kAhead = KB < 3 ? KB : 3;
    for (; blk < nblk; blk += WAVES) {
        // float16 norms of the lane's 16 result rows per tile: four runs of four consecutive vectors
        uint32_t cg[S][8];
        const uint16_t* gb = a.store.gamma + t.base_slot + v_lo + blk * VB + 4 * half;
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const uint2 two = *reinterpret_cast<const uint2*>(gb + 32 * s + 8 * g);
                cg[s][2 * g] = two.x;
                cg[s][2 * g + 1] = two.y;
            }
        // de-quantise: coordinates 16*kb + 8*half + [0, 8) of vector jl of either tile
        half8 ah[S][KB];
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const uint64_t chunk = code_chunk<B, NW>(cw[s][kb], kb, half);
                uint32_t hv[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (Cfg::PAIR) {
                        hv[i] = mine[((uint32_t)(chunk >> (2 * B * i)) & (uint32_t)(Cfg::PT - 1)) * TC];
                    } else {
                        const uint32_t e0 = mine[((uint32_t)(chunk >> (2 * B * i)) & (uint32_t)(Cfg::PT - 1)) * TC];
                        const uint32_t e1 = mine[((uint32_t)(chunk >> (2 * B * i + B)) & (uint32_t)(Cfg::PT - 1)) * TC];
                        hv[i] = e0 | (e1 << 16);
                    }
                }
                ah[s][kb] = __builtin_bit_cast(half8, make_uint4(hv[0], hv[1], hv[2], hv[3]));
            }
        // the next block's words, whose registers are free now, travel while this one is multiplied
        if (blk + WAVES < nblk) fetch(blk + WAVES);
        if (v_lo + blk * VB + VB > v_hi) {
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int v = v_lo + blk * VB + 32 * s + 8 * (r / 4) + 4 * half + (r % 4);
                    if (v >= v_hi) cg[s][r / 2] = (r & 1) ? ((cg[s][r / 2] & 0xFFFFu) | 0x7E000000u) : ((cg[s][r / 2] & 0xFFFF0000u) | 0x7E00u);
                }
        }
        // the largest norm among this lane's rows (packed float16 maxima, which skip the NaNs), for a raw metric
        // also the range of the vectors' lengths
        typedef _Float16 half2v __attribute__((ext_vector_type(2)));
        float g_max[S], x_min[S], x_max[S];
#pragma unroll
        for (int s = 0; s < S; ++s) {
            half2v gm = __builtin_bit_cast(half2v, cg[s][0]);
#pragma unroll
            for (int r = 1; r < 8; ++r) gm = __builtin_elementwise_max(gm, __builtin_bit_cast(half2v, cg[s][r]));
            g_max[s] = kUnscale * fmaxf((float)gm[0], (float)gm[1]);
            x_min[s] = __builtin_inff();
            x_max[s] = 0.f;
            if (RAW) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int v = v_lo + blk * VB + 32 * s + 8 * (r / 4) + 4 * half + (r % 4);
                    const float xn = a.store.xnorm[t.base_slot + (v < v_hi ? v : v_hi - 1)];
                    x_min[s] = fminf(x_min[s], xn);
                    x_max[s] = fmaxf(x_max[s], xn);
                }
            }
        }
        // No row of a tile can reach the threshold unless the largest accumulator times the largest norm
        // does: g_max >= g_r >= 0 and a_max >= max(acc_r, 0), and a correctly rounded sum or fused multiply-add never
        // decreases when its exact value grows, so fmaf(g_max, a_max + acc0, sq) >= fmaf(g_r, acc_r + acc0, sq).
        auto take = [&](const floatx16& acc, int s, int qt) {
            const uint4 row = s_row[qt * 32 + jl];
            const float sq = __uint_as_float(row.x), th = __uint_as_float(row.y);
            float a_max = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 2) a_max = fmaxf(fmaxf(a_max, acc[r]), acc[r + 1]);
            float top = fmaf(g_max[s], a_max + a.acc0, sq);
            if (RAW) top = metric_key_bound(a.metric, top, x_min[s], x_max[s], __uint_as_float(row.w));
            if (top >= th) {                       // seldom: some row of this lane may reach the threshold
                // (the first row's number is hidden from the compiler, which would otherwise prepare every row's
                // addresses ahead of the tiles and spill them)
                int v0 = v_lo + blk * VB + 32 * s + 4 * half;
                asm volatile("" : "+v"(v0));
                auto key_of = [&](int r) -> float {
                    uint32_t two = cg[s][r / 2];
                    asm volatile("" : "+v"(two));   // likewise converted where it is read
                    const float g = kUnscale * __half2float(__ushort_as_half((uint16_t)((r & 1) ? (two >> 16) : (two & 0xFFFFu))));
                    float u = fmaf(g, acc[r] + a.acc0, sq);  // upper bound of the score; NaN never passes
                    if (RAW) {
                        const int v = v0 + 8 * (r / 4) + (r % 4);
                        u = metric_key(a.metric, u, a.store.xnorm[t.base_slot + (v < v_hi ? v : v_hi - 1)], __uint_as_float(row.w));
                    }
                    return u;
                };
                // counted first: one update of the query's counter for all of the lane's rows (its latency, once per
                // row, was 2/3 of the pass where 1 in 80 vectors is appended)
                uint32_t hit = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) hit |= key_of(r) >= th ? 1u << r : 0u;
                if (hit) {
                    const int n_hit = (int)__popc(hit);
                    int held = CAND;
                    if (HOLD) held = atomicAdd(&s_next[2], n_hit);
                    if (HOLD && held + n_hit <= CAND) {
                        const int e = qt * 32 + jl;
                        uint32_t word = (uint32_t)(e | (v0 - v_lo) << 7) + ((uint32_t)atomicAdd(&s_cnt[e], n_hit) << 19);
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if ((hit >> r) & 1u) {
                                s_cand[held++] = make_uint2(__float_as_uint(key_of(r)), word + ((uint32_t)(8 * (r / 4) + (r % 4)) << 7));
                                word += 1u << 19;
                            }
                    } else {
                        if (HOLD) atomicMin(&s_next[3], held);
                        const int32_t q = (int32_t)row.z / a.np;
                        const int64_t rank = (int64_t)((int32_t)row.z - q * a.np) << kCandProbeShift;
                        const int pos = atomicAdd(&a.cand_cnt[q], n_hit);
                        const int room = a.cap - pos;
                        float* to_score = a.cand_score + (int64_t)q * a.cap + pos;
                        int64_t* to_slot = a.cand_slot + (int64_t)q * a.cap + pos;
                        const int64_t slot0 = (t.base_slot + v0) | rank;       // adding to the slot stays below the rank
                        int at = 0;
#pragma unroll
                        for (int r = 0; r < 16; ++r)
                            if ((hit >> r) & 1u) {
                                if (at < room) {
                                    to_score[at] = key_of(r);
                                    to_slot[at] = slot0 + 8 * (r / 4) + (r % 4);
                                }
                                ++at;
                            }
                    }
                }
            }
        };
        for (int qt = 0; qt < n_qt; ++qt) {
            const uint16_t* b0 = bh_base + qt * 32 * Cfg::LDH;
            floatx16 acc[S];
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[s][r] = 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const half8 h = *reinterpret_cast<const half8*>(b0 + 16 * kb);
#pragma unroll
                for (int s = 0; s < S; ++s) acc[s] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah[s][kb], h, acc[s], 0, 0, 0);
            }
            // the panel reads run kAhead blocks ahead of the products (the compiler's own order, each read right before
            // its products, leaves the LDS latency exposed once per block)
            __builtin_amdgcn_sched_group_barrier(0x100, kAhead + 1, 0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                __builtin_amdgcn_sched_group_barrier(0x008, S, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
#pragma unroll
            for (int s = 0; s < S; ++s) take(acc[s], s, qt);
        }
    }
    }
}

template <int DP, int B>
hipError_t run_batch(const BatchScanArgs& a, hipStream_t st) {
    static ChipFill fill;
    if (a.dense) {
        constexpr int NQ = kBatchTileNear / 32;
        constexpr size_t lds = BatchCfg<DP, B, NQ>::lds_dense;
        constexpr auto dense = k_batch_dense<DP, B, NQ, 4, 2>;
        unsigned wgs = 0;
        const hipError_t e = fill.get(reinterpret_cast<const void*>(dense), 256, lds, &wgs);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(dense, dim3(wgs), dim3(256), lds, st, a);
    } else {
        static ChipFill fill_t[3];
        constexpr int NQ = kBatchTile / 32;
        // two row tiles and wavefronts per SIMD where the registers (operands of both tiles, and the words of the
        // next block, twice or four times as many where codes straddle words or are bytes) allow it without spills
        constexpr int words = B == 8 ? DP / 4 : (B == 3 || B == 5) ? DP / 8 : DP / 16;
        constexpr int S = DP + 2 * words <= 256 ? 2 : 1, S_RAW = DP + 2 * words < 200 ? 2 : 1;
        constexpr int OCC = S == 2 && DP + words <= 102 ? 3 : 2;
        constexpr bool HOLD = OCC == 2 || DP <= 64;
        using Cfg = BatchCfg<DP, B, NQ>;
        // Copies of the table (4 bits: 256 entries; a table of 64 has no two entries on one bank, one of 1024 leaves too little
        // room): a workgroup makes them once, 1 to 2 us, which only a long pass pays back, and they take room from the candidates held
        // back, which rows without clusters need.  So where the pass is long and what such rows would leave in a tile fits all
        // the same.  Pass with copies and without, us, 64 probes of 3M x 200: 256 queries 124 and 129, 10,000 474 and 495; 32 of 3M x 96:
        // 256 queries 88 and 86, 10,000 148 and 150; 24 of 400,000 x 128: 300 queries 27.5 and 26.4; 400,000 rows without clusters,
        // 4000 queries, k = 100: x 192 266 and 218, x 208 295 and 222, x 224 340 and 250.
        constexpr bool kCopied = B == 4 && Cfg::copies_fit(OCC, HOLD);
        constexpr int TC = kCopied ? kTableCopies : 1;
        const bool copied = kCopied && !a.metric && a.dequantised >= kCopiesFrom && (!HOLD || a.tile_candidates <= Cfg::held_back(OCC, TC));
        constexpr auto plain = k_batch_threshold<DP, B, NQ, 4, OCC, S, false, HOLD, 1>, with_copies = k_batch_threshold<DP, B, NQ, 4, OCC, S, false, HOLD, TC>;
        constexpr auto raw = k_batch_threshold<DP, B, NQ, 4, 2, S_RAW, true, true, 1>;
        const auto go = [&](ChipFill& fill, auto kernel, size_t lds) -> hipError_t {
            unsigned wgs = 0;
            const hipError_t e = fill.get(reinterpret_cast<const void*>(kernel), 256, lds, &wgs);
            if (e == hipSuccess) hipLaunchKernelGGL(kernel, dim3(wgs), dim3(256), lds, st, a);
            return e;
        };
        const hipError_t e = a.metric ? go(fill_t[1], raw, Cfg::lds_threshold(2, true, 1))
                             : copied ? go(fill_t[2], with_copies, Cfg::lds_threshold(OCC, HOLD, TC))
                                      : go(fill_t[0], plain, Cfg::lds_threshold(OCC, HOLD, 1));
        if (e != hipSuccess) return e;
    }
    return hipGetLastError();
}

template <int B>
hipError_t run_batch_width(const BatchScanArgs& a, int dp, hipStream_t st) {
    switch (dp) {
        case 64: return run_batch<64, B>(a, st);
        case 96: return run_batch<96, B>(a, st);
        case 128: return run_batch<128, B>(a, st);
        case 160: return run_batch<160, B>(a, st);
        case 192: return run_batch<192, B>(a, st);
        case 208: return run_batch<208, B>(a, st);
        case 224: return run_batch<224, B>(a, st);
        case 256: return run_batch<256, B>(a, st);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace

}  // namespace ivftq
