// The kernel of the query-batched list scan, one instantiation per (panel width, stored bits); included by the
// translation units batch_scan_b*.hip, which compile the widths of one bit count each.
//
// A wavefront takes a part of one list and up to TQ of the queries that probe it.  The rotated queries are one MFMA operand and stay in
// registers (but for what some wide forms spill, see batch_query_tiles); the vectors, 32 at a time, are the other, de-quantised through a table in LDS block by block into the products that use
// them.
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
// v_mfma_f32_16x16x32_f16: A is 16x32 (lane = i + 16*(k/8), element k%8), B likewise, D[i][j] in lane j + 16*(i/4), register i%4.
#pragma once
#include <hip/hip_fp16.h>

#include <type_traits>

#include "kernels.h"

namespace ivftq {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef _Float16 half8 __attribute__((ext_vector_type(8)));

namespace {

// Table of code pairs (2^(2b) entries of two levels; 8 bits: of single codes) that de-quantises, in as many copies as spare a look-up's
// lanes all collisions on banks (a copy for each of the 64 lanes, or for the 32 that an 8-byte read serves at a time), or as fit.  A
// compute unit holds one workgroup of all its wavefronts, which share the table.  Entry e's copies lie in a row of STRIDE bytes, so that
// where an index is a byte of the codes (4 and 8 bits) and a row 256 bytes, an address is one byte permutation of codes and lane.
template <int B, bool BOTH>
struct Table {
    static constexpr bool PAIR = B <= 5;                          // two codes per look-up
    static constexpr int BITS = PAIR ? 2 * B : B, PT = 1 << BITS;
    static constexpr int ENTRY = PAIR && BOTH ? 8 : 4;            // bytes: (hi pair, lo pair) or hi pair; one code: hi | lo << 16
    static constexpr int STRIDE = PT * 256 <= 64 * 1024 ? 256 : 64 * 1024 / PT;
    static constexpr int TC = STRIDE / ENTRY, BYTES = PT * STRIDE;

    // by all threads of a workgroup; a barrier has to follow
    static __device__ __forceinline__ void fill(unsigned char* to, const float* cb, int threads) {
        constexpr int kPieces = STRIDE / 16;
        for (int p = threadIdx.x; p < PT * kPieces; p += threads) {
            const int e = p / kPieces;
            uint32_t hp = 0, lp = 0;
#pragma unroll
            for (int i = 0; i < (PAIR ? 2 : 1); ++i) {
                const float V = cb[(e >> (i * B)) & ((1 << B) - 1)] * kSplitScale;
                const _Float16 hi = (_Float16)V;
                const _Float16 lo = (_Float16)(V - (float)hi);
                hp |= (uint32_t)__builtin_bit_cast(uint16_t, hi) << (16 * i);
                lp |= (uint32_t)__builtin_bit_cast(uint16_t, lo) << (16 * i);
            }
            if (!PAIR) hp |= BOTH ? lp << 16 : 0u;
            *reinterpret_cast<uint4*>(to + p * 16) = ENTRY == 8 ? make_uint4(hp, lp, hp, lp) : make_uint4(hp, hp, hp, hp);
        }
    }
    // byte offset of the entry at bit `bit` of the codes, in the copy that begins at byte `own` of a row
    static __device__ __forceinline__ uint32_t at(uint64_t codes, int bit, uint32_t own) {
        if constexpr (BITS == 8 && STRIDE == 256)
            return __builtin_amdgcn_perm((uint32_t)(codes >> (bit & 32)), own, 0x0C0C0000u | (uint32_t)(4 + bit % 32 / 8) << 8);
        else
            return ((uint32_t)(codes >> bit) & (uint32_t)(PT - 1)) * STRIDE + own;
    }
    // The entries of the 8 codes of a lane, as they come from LDS ...
    struct Raw { uint32_t w[PAIR && !BOTH ? 4 : 8]; };
    static __device__ __forceinline__ void look_up(const unsigned char* table, uint32_t own, uint64_t codes, Raw& r) {
        if constexpr (PAIR && BOTH) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint2 e = *reinterpret_cast<const uint2*>(table + at(codes, 2 * B * i, own));
                r.w[2 * i] = e.x;
                r.w[2 * i + 1] = e.y;
            }
        } else {
#pragma unroll
            for (int i = 0; i < (PAIR ? 4 : 8); ++i) r.w[i] = *reinterpret_cast<const uint32_t*>(table + at(codes, (PAIR ? 2 : 1) * B * i, own));
        }
    }
    // ... and as operands: both parts (BOTH) or the leading ones.  (hi, lo) of one pair and of the next become (hi, hi) and (lo, lo) by
    // an exchange, so that four registers in a row are an operand.  A matrix instruction must not follow a write of its operands by fewer
    // than two states; the compiler does not look into assembly for that, so the wait belongs to the exchange.  (By value: with the entries of
    // a block that is looked up once in a slab, exchanged in place through a reference, the compiler kept them in scratch memory.)
    static __device__ __forceinline__ void operands(Raw r, half8& hi, half8& lo) {
        if constexpr (PAIR && BOTH) {
            asm("v_swap_b32 %0, %1\n\tv_swap_b32 %2, %3\n\ts_nop 1" : "+v"(r.w[1]), "+v"(r.w[2]), "+v"(r.w[5]), "+v"(r.w[6]));
            hi = __builtin_bit_cast(half8, make_uint4(r.w[0], r.w[1], r.w[4], r.w[5]));
            lo = __builtin_bit_cast(half8, make_uint4(r.w[2], r.w[3], r.w[6], r.w[7]));
        } else if constexpr (PAIR) {
            hi = __builtin_bit_cast(half8, make_uint4(r.w[0], r.w[1], r.w[2], r.w[3]));
        } else {
            uint32_t hv[4], lv[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                hv[i] = __builtin_amdgcn_perm(r.w[2 * i + 1], r.w[2 * i], 0x05040100u);
                lv[i] = __builtin_amdgcn_perm(r.w[2 * i + 1], r.w[2 * i], 0x07060302u);
            }
            hi = __builtin_bit_cast(half8, make_uint4(hv[0], hv[1], hv[2], hv[3]));
            if (BOTH) lo = __builtin_bit_cast(half8, make_uint4(lv[0], lv[1], lv[2], lv[3]));
        }
    }
};

// Wavefronts of a workgroup, which has a compute unit to itself, and its LDS.
constexpr int waves_of(int per_simd) { return 4 * per_simd; }
constexpr size_t kLdsRoom = 160 * 1024;

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
    int v_lo, v_hi, nq_tile;             // vectors [v_lo, v_hi) of a list; v_lo is a multiple of 64
    int pair0;
    int64_t base_slot;
    // size, ...: of the record of the tile's bucket
    __device__ __forceinline__ void set(int tile, int part_len, int tq, int size, int first_tile, int count, int first_pair, int slot_lo, int slot_hi) {
        const int parts = list_parts(size, part_len), rel = tile - first_tile;
        const int len = ((size + parts - 1) / parts + 63) & ~63;
        v_lo = (rel % parts) * len;
        v_hi = v_lo + len < size ? v_lo + len : size;
        const int skip = rel / parts * tq, left = count - skip;
        pair0 = first_pair + skip;
        nq_tile = left < tq ? left : tq;
        base_slot = (int64_t)(((uint64_t)(uint32_t)slot_hi << 32) | (uint32_t)slot_lo);
    }
};

// The workgroups of a launch are as many as the chip holds and every wavefront takes tiles of its own until none is left, the first two
// by its number, the others from the counter of its workgroup's queue: tiles differ in work by the sizes of the lists and the queries that
// meet there.  No wavefront waits for another (with a tile to a workgroup, whose wavefronts met at a barrier and waited for the counter,
// half of all wavefront cycles went by waiting).  Finding a tile's bucket, record, pairs and queries is a chain of five dependent reads of
// 0.7 us and more; most are made while the tiles before it are worked on: its number is asked for two tiles ahead, its bucket
// one tile ahead, the record after slab 2 of the tile before and the pairs after its slab 8.  A tile of 256 vectors, which most have, has slabs 0 to 7,
// so there the pairs are read between the tiles.  What is asked for comes behind the words of vectors on their way, so the wait for it is one for
// those too.
// TQ: queries of a tile.
template <int TQ>
struct TileQueue {
    const BatchScanArgs& a;
    const int32_t* bucket_of;
    int32_t* counter;
    BatchTile t;                         // the tile to work on
    int tile, end;                       // its number (past `end`: none)
    int next, asked, q, given;           // queue, and its tiles given by number
    int phase = 0;                       // of the next tile: 0 its bucket asked for, 1 its record, 2 its pairs
    int32_t known[(TQ + 63) / 64];       // in turn its bucket, its record, the pairs of queries lane and 64 + lane
    BatchTile tn;
    __device__ __forceinline__ TileQueue(const BatchScanArgs& args, int wave, int waves) : a(args) {
        bucket_of = a.dense ? a.p.tile_near : a.p.tile_late;
        end = a.p.totals[a.dense ? 1 : 2];
        q = (int)blockIdx.x % kTileQueues;
        counter = a.p.totals + 32 + ((a.dense ? 0 : kTileQueues) + q) * 32;
        const int servers = queue_servers((int)gridDim.x, q) * waves;        // wavefronts
        const int me = (int)blockIdx.x / kTileQueues * waves + wave;
        given = 2 * servers;
        next = queue_tile(q, me);
        asked = servers + me - given;    // (the second tile by number, as if asked for)
        if (next < end) known[0] = bucket_of[next];
        advance();
    }
    // (through registers of the lanes' own, or the compiler waits for the answers where they are asked for)
    __device__ __forceinline__ void ask() {
        int lane = (int)(threadIdx.x & 63);
        asm volatile("" : "+v"(lane));
        if (lane == 0) {
            asked = atomicAdd(counter + lane, 1);
            known[0] = bucket_of[(next < end ? next : 0) + lane];
        }
    }
    // between slabs
    __device__ __forceinline__ void between(int slab) {
        if (slab == 2 || slab == 8) step();
    }
    __device__ __forceinline__ void step() {
        if (phase >= 2 || next >= end) return;
        int lane = (int)(threadIdx.x & 63);
        asm volatile("" : "+v"(lane));
        if (phase++ == 0) {
            known[0] = (a.p.record + (int64_t)__builtin_amdgcn_readfirstlane(known[0]) * kPairRecord)[lane & (kPairRecord - 1)];
        } else {
            auto word = [&](int i) { return __builtin_amdgcn_readlane(known[0], i); };
            tn.set(next, a.part_len, TQ, word(0), word(1), word(2), word(3), word(4), word(5));
#pragma unroll
            for (int i = 0; i < (TQ + 63) / 64; ++i) known[i] = (a.p.pairs + tn.pair0)[min(64 * i + lane, tn.nq_tile - 1)];
        }
    }
    __device__ __forceinline__ void advance() {
        while (phase < 2 && next < end) step();
        tile = next;
        t = tn;
        next = queue_tile(q, __builtin_amdgcn_readfirstlane(asked) + given);
        phase = 2;
    }
    // pair of query e of the tile (some other one beyond its last); before `proceed`
    __device__ __forceinline__ int32_t pair_of(int e) const {
        int32_t p = __shfl(known[0], e & 63);
        if (TQ > 64 && e >= 64) p = __shfl(known[(TQ + 63) / 64 - 1], e & 63);
        return p;
    }
    // once the tile's pairs are no longer asked for
    __device__ __forceinline__ void proceed() {
        phase = 0;
        ask();
    }
};

// What a wavefront's lanes left in LDS is there for its other lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A wavefront's operand of the tile's queries: lane jl of either half takes the coordinates 16 kb + 8 half + [0, 8) of its query, whose
// split row begins at `row`.  (Beyond a tile's last query some other one, whose results are not looked at.)
template <int DP>
__device__ __forceinline__ void load_query(const uint16_t* row, int z_pitch, half8 (&out)[DP / 16]) {
#pragma unroll
    for (int kb = 0; kb < DP / 16; ++kb) {
        out[kb] = half8{};
        if (DP > 64 || 16 * kb < z_pitch) out[kb] = *reinterpret_cast<const half8*>(row + 16 * kb);       // (rows are as wide as wider panels)
    }
}

// A lane's offset as the compiler is to take it where it is used: made 64 bits wide, or scaled, ahead of a loop it is spilled.
__device__ __forceinline__ uint32_t lane_offset(int v) {
    asm volatile("" : "+v"(v));
    return (uint32_t)v;
}

// The packed words of a slab of 32 vectors: lane jl of either half takes its vector's codes 16 kb + 8 half + [0, 8), which begin in word
// first_word(kb, half).  The upper half's words lie a fixed 0, 1 or 2 words after the lower half's, so a load is a wavefront's address, a
// lane's offset for each such distance, and a constant.  Only in the last blocks, which a row of the fewest coordinates of this panel does
// not fill, is the word's number bounded by the row's: what is read there in place of a word that does not exist meets zero coordinates.
template <int DP, int B, int NW>
struct SlabWords {
    static constexpr int KB = DP / 16;
    static constexpr int least = DP <= 64 ? 16 : DP == 224 ? 209 : DP == 208 ? 193 : DP - 31;      // fewest coordinates
    static constexpr int sure = (B * least + 31) / 32;            // words that every row has
    int words, half, jl;
    __device__ __forceinline__ void load(const uint32_t* slab, int kb, uint32_t (&w)[NW]) const {
        const int w0 = first_word<B>(kb, 0), step = first_word<B>(kb, 1) - w0;
#pragma unroll
        for (int e = 0; e < NW; ++e) {
            if (w0 + step + e < sure) w[e] = (slab + (w0 + e) * 64)[(uint32_t)(64 * step * half + jl)];
            else {
                const uint32_t at = lane_offset(64 * step * half + jl);
                w[e] = slab[min(at + (uint32_t)(w0 + e) * 64, (at & 63) + (uint32_t)(words - 1) * 64)];
            }
        }
    }
};

// ---- dense pass: every score of the nearest lists is stored -------------------------------------------
//
// A list is among the nearest of few queries (three at 10M x 96 with 10,000 queries, eleven at 10M x 200), so tiles of 16 queries are
// multiplied, up to two of them a tile of the pass.  The queries are the row operand, held in registers for the whole tile, and the vectors, two
// groups of 16 to a slab, the column operand, de-quantised block by block into the products that use them, so that LDS serves
// nothing but the look-ups.  A lane holds a vector's scores against every fourth query, so that a tile of at most four queries, rows 0, 4, 8
// and 12, stores 64 bytes of each with one instruction.
// Bound by memory: at 10M x 96 (10,000 queries, 32 probes) the pass reads 0.52 GB and writes 0.12 in 147 to 150 us, 4.3 TB/s where a large copy
// moves 4.8; at 10M x 200 (64 probes, k = 100) 1.48 and 0.54 GB in 402 to 409 us, 5.0 TB/s.  With the queries in LDS, 32 x 32 products, a tile to
// a workgroup and one counter for all tiles 240 and 610 us.
// RAW: scores are ranking keys of a raw metric.
typedef float floatx4 __attribute__((ext_vector_type(4)));

// The packed words of 16 vectors: lane 16 h + j takes vector j's codes 32 kb + 8 h + [0, 8), from bit 8 h B of block kb's words on.
template <int DP, int B, int NW>
struct GroupWords {
    static constexpr int least = DP <= 64 ? 16 : DP == 224 ? 209 : DP == 208 ? 193 : DP - 31;      // fewest coordinates
    static constexpr int sure = (B * least + 31) / 32;            // words that every row has
    int words, own;                                               // own: place of the lane's first word and vector in a block
    __device__ __forceinline__ GroupWords(int row_words, int lane) : words(row_words), own(((lane >> 4) * B >> 2) * 64 + (lane & 15)) {}
    __device__ __forceinline__ void load(const uint32_t* group, int kb, uint32_t (&w)[NW]) const {
        constexpr int last = 3 * B >> 2;
#pragma unroll
        for (int e = 0; e < NW; ++e) {
            if (kb * B + last + e < sure) w[e] = (group + (kb * B + e) * 64)[(uint32_t)own];
            else {
                const uint32_t at = lane_offset(own);
                w[e] = group[min(at + (uint32_t)(kb * B + e) * 64, (at & 63) + (uint32_t)(words - 1) * 64)];
            }
        }
    }
    __device__ __forceinline__ uint64_t codes(const uint32_t (&w)[NW], int lane) const {
        const int bit = (lane >> 4) * 8 * B & 31;
        if constexpr (NW == 1) return B == 4 ? w[0] : w[0] >> bit;
        else return B == 8 ? ((uint64_t)w[1] << 32) | w[0] : (((uint64_t)w[1] << 32) | w[0]) >> bit;
    }
};

// About the registers that the dense pass takes for n row tiles of queries (operands, accumulators, places), blocks in flight, and words of
// `ahead` slabs.  (256 coordinates of 8 bits spill 27 registers, 65 with a raw metric, 3, 5 and other 8-bit forms up to 15.)
constexpr int dense_registers(int dp, int b, bool raw, int n, int ahead) {
    const int kb = (dp + 31) / 32, nw = b == 2 || b == 4 ? 1 : 2;
    return n * (8 * kb + 8 + (raw ? 16 : 12)) + 32 + ahead * (2 * kb * nw + (raw ? 4 : 2)) + 38;
}

template <int DP, int B, bool RAW>
struct DenseCfg { static constexpr int OCC = dense_registers(DP, B, RAW, 2, 1) <= 168 ? 3 : 2; };

template <int DP, int B, bool RAW>
__global__ __launch_bounds__(64 * waves_of(DenseCfg<DP, B, RAW>::OCC)) __attribute__((amdgpu_waves_per_eu(DenseCfg<DP, B, RAW>::OCC)))
void k_batch_dense(BatchScanArgs a) {
    using Tab = Table<B, true>;
    constexpr int OCC = DenseCfg<DP, B, RAW>::OCC;
    constexpr int KB = (DP + 31) / 32, TQ = kBatchTileNear, WAVES = waves_of(OCC);
    constexpr int NW = (B == 2 || B == 4) ? 1 : 2;
    static_assert(TQ == 32, "two row tiles of queries");
    typedef __attribute__((address_space(1))) float global_float;
    extern __shared__ __align__(16) unsigned char table[];

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, quarter = lane >> 4, jl = lane & 15;
    constexpr float kUnscale = 1.f / (kSplitScale * kSplitScale);

    Tab::fill(table, a.cb, 64 * WAVES);
    const uint32_t own = (uint32_t)(tid % Tab::TC * Tab::ENTRY);
    const int words = a.store.words;
    const GroupWords<DP, B, NW> from(words, lane);
    __syncthreads();
    for (TileQueue<TQ> queue(a, wave, WAVES); queue.tile < queue.end; queue.advance()) {
    const BatchTile t = queue.t;
    const int n_v = t.v_hi - t.v_lo, nslab = (n_v + 31) / 32;
    // A list starts at a multiple of 64 slots and its slots reach to one, so a slab's words and norms can be read whole.
    const uint32_t* codes = a.store.codes + ((t.base_slot + t.v_lo) >> 6) * words * 64;
    const uint16_t* norms = a.store.gamma + t.base_slot + t.v_lo;
    const float* lengths = RAW ? a.store.xnorm + t.base_slot + t.v_lo : nullptr;
    auto slab_at = [&](int slab) { return codes + (int64_t)(slab >> 1) * words * 64 + (slab & 1) * 32; };

    auto scan_tile = [&](auto tiles) {
        constexpr int N = decltype(tiles)::value;
        // Words and norms of a slab on their way: two slabs ahead of the products, or one where the registers do not reach for two.
        // (After every AHEAD slabs the compiler waits for all that is on its way, to move the last norm to another register.)
        constexpr int AHEAD = dense_registers(DP, B, RAW, N, 2) <= (OCC == 3 ? 168 : 256) ? 2 : 1;
        struct Ahead { uint32_t w[2][KB][NW], g16[2]; float xn[2]; } ahead[AHEAD];
        auto fetch_norms = [&](int slab, Ahead& f) {
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                f.g16[c] = (norms + slab * 32 + 16 * c)[lane_offset(jl)];
                if (RAW) f.xn[c] = (lengths + slab * 32 + 16 * c)[lane_offset(jl)];
            }
        };
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int slab = i < nslab ? i : 0;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int c = 0; c < 2; ++c) from.load(slab_at(slab) + 16 * c, kb, ahead[i].w[c][kb]);
            fetch_norms(slab, ahead[i]);
        }
        half8 qh[N][KB], ql[N][KB];
        // of the lane's queries 16 n + 4 i + quarter: coarse term, place of the score of the part's first vector, |q| (RAW)
        float coarse[N][4], qn[N][4];
        global_float* to[N][4];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int64_t row = (int64_t)(queue.pair_of(16 * n + 4 * (jl % 4) + jl / 4) / a.np) * a.z_pitch + 8 * quarter;      // (row 4 h + i: query 4 i + h)
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                qh[n][kb] = ql[n][kb] = half8{};
                if (DP > 64 || 32 * kb < a.z_pitch) {              // (rows are as wide as wider panels)
                    qh[n][kb] = *reinterpret_cast<const half8*>(a.zh + row + 32 * kb);
                    ql[n][kb] = *reinterpret_cast<const half8*>(a.zl + row + 32 * kb);
                }
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int32_t it = queue.pair_of(16 * n + 4 * i + quarter), q = it / a.np;
                coarse[n][i] = a.coarse[it];
                to[n][i] = (global_float*)(a.scores + (int64_t)q * a.m_stride + a.cand_off[(int64_t)q * (a.np + 1) + (it - q * a.np)] + t.v_lo);
                qn[n][i] = RAW ? a.qnorm[q] : 0.f;
            }
        }
        queue.proceed();

        auto scan = [&](int slab, Ahead& f) {
            // A block's words make room for those of the same block AHEAD slabs on as soon as they are looked up.
            const int next = slab + AHEAD < nslab ? slab + AHEAD : slab;
            const uint32_t* next_at = slab_at(next);
            typename Tab::Raw raw[2][2];             // blocks in flight: one ahead of the products
            auto look = [&](int kb) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    Tab::look_up(table, own, from.codes(f.w[c][kb], lane), raw[kb % 2][c]);
                    from.load(next_at + 16 * c, kb, f.w[c][kb]);
                }
            };
            look(0);
            floatx4 acc[2][N];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int n = 0; n < N; ++n) acc[c][n] = floatx4{0.f, 0.f, 0.f, 0.f};
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb + 1 < KB) look(kb + 1);
                half8 vh[2], vl[2];
#pragma unroll
                for (int c = 0; c < 2; ++c) Tab::operands(raw[kb % 2][c], vh[c], vl[c]);
                auto product = [&](const half8 (&q)[N][KB], const half8 (&v)[2]) {
#pragma unroll
                    for (int n = 0; n < N; ++n)
#pragma unroll
                        for (int c = 0; c < 2; ++c) acc[c][n] = __builtin_amdgcn_mfma_f32_16x16x32_f16(q[n][kb], v[c], acc[c][n], 0, 0, 0);
                };
                product(qh, vh);
                product(ql, vh);
                product(qh, vl);
                __builtin_amdgcn_sched_barrier(0);
            }
            float g[2], xn[2];
            bool in_part[2];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                g[c] = kUnscale * __half2float(__ushort_as_half((uint16_t)f.g16[c]));      // 2^-20 * norm of this lane's vector
                xn[c] = RAW ? f.xn[c] : 0.f;
                in_part[c] = slab * 32 + 16 * c + jl < n_v;
            }
            fetch_norms(next, f);
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (16 * n + 4 * i >= t.nq_tile) break;       // (a sparse tile skips the fours it has no query for)
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        float sc = fmaf(g[c], acc[c][n][i], coarse[n][i]);
                        if (RAW) sc = metric_key(a.metric, sc, xn[c], qn[n][i]);
                        if (16 * n + 4 * i + quarter < t.nq_tile && in_part[c]) to[n][i][slab * 32 + 16 * c + jl] = sc;
                    }
                }
        };
        for (int slab = 0; slab < nslab; slab += AHEAD) {
            scan(slab, ahead[0]);
            if (AHEAD > 1 && slab + 1 < nslab) scan(slab + 1, ahead[AHEAD - 1]);
            queue.between(slab);
        }
    };
    if (t.nq_tile > 16) scan_tile(std::integral_constant<int, 2>{});
    else scan_tile(std::integral_constant<int, 1>{});
    }
}

// The largest of the 32 numbers that the lanes of either half hold (the halves hold the same), in every lane.
__device__ __forceinline__ int slab_max(int v) {
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x128, 0xf, 0xf, true));        // row_ror:8, 4, 2, 1
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x124, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x122, 0xf, 0xf, true));
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x121, 0xf, 0xf, true));
    const auto r = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    const unsigned r0 = r[0], r1 = r[1];
    return max((int)r0, (int)r1);
}

// ---- threshold pass: the other lists, only scores that can reach the query's threshold kept ------------
//
// The vectors are the row operand, so a lane holds one query's scores against 16 vectors and needs that query's
// coarse term and threshold only once.  Only the leading float16 parts are multiplied (one product instead of
// three): acc0 = 2^20 * kappa is added to the accumulators, kappa bounding the error of such a sum for a unit query,
// so what is compared with the threshold and appended is an upper bound of the true score (true score in
// [u - 2*kappa*gamma, u]); k_merge re-scores from the packed codes the few that can still matter.
//
// The queries, up to NQ tiles of 32, are held in registers, so that LDS serves nothing but the look-ups: a block of 16 coordinates of 32
// vectors is de-quantised (4 look-ups, 8 LDS clocks shared by four SIMDs) into NQ matrix instructions (32 clocks each).  At 10M x 200 (10,000
// queries, 64 probes) the matrix pipe is busy half of the cycles, at the 1.8 GHz the chip holds under this load: 765 to 795 us, where queries in
// LDS, read for every product, took 870; at 10M x 96 (32 probes) 235 to 240 us, a third of the cycles: the rest goes into finding tiles, and what a
// slab and a row tile take besides their products.
// RAW: scores are ranking keys of a raw metric.
//
// A candidate is appended to its query's list with an update of the query's counter, whose answer its stores wait for.  Where candidates
// are many and queries few, such updates are what the pass takes.  So the candidates of a tile are held back in LDS and a counter is updated once per tile (rows without clusters, 1M x
// 128, inner product, 100 queries of 64 probes, k = 100, up to 1172 candidates a query: 203 -> 104 us); what does not fit is
// appended at once.
template <int DP, int B, int NQ, int OCC>
struct ThresholdCfg {
    using Tab = Table<B, false>;
    static constexpr int TQ = NQ * 32;
    static constexpr int WAVES = waves_of(OCC);
    static constexpr size_t own = (16 + 4) * TQ + 2 * 32 * sizeof(float) + 2 * sizeof(int);         // of a wavefront, besides what it holds back
    static constexpr int fit = (int)((kLdsRoom - Tab::BYTES - WAVES * own) / (8 * WAVES)), CAND = fit < 1024 ? fit / 2 * 2 : 1024;      // candidates held back
    static constexpr size_t lds = Tab::BYTES + WAVES * (own + 8 * (size_t)CAND);
    static_assert(CAND >= 200 && TQ <= 128 && kPartMax <= 4096, "fields of a candidate held back");
};

template <int DP, int B, int NQ, int OCC, bool RAW>
__global__ __launch_bounds__(64 * waves_of(OCC)) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_batch_threshold(BatchScanArgs a) {
    using Cfg = ThresholdCfg<DP, B, NQ, OCC>;
    using Tab = typename Cfg::Tab;
    constexpr int KB = DP / 16, TQ = Cfg::TQ, CAND = Cfg::CAND, WAVES = Cfg::WAVES;
    constexpr int NW = (B == 2 || B == 4) ? 1 : 2;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, jl = lane & 31;
    extern __shared__ __align__(16) unsigned char table[];
    // (everything behind the table is a wavefront's own)
    uint4* s_row = reinterpret_cast<uint4*>(table + Tab::BYTES) + wave * TQ;                    // [TQ] coarse term, threshold, pair number, |q|
    uint2* s_cand = reinterpret_cast<uint2*>(table + Tab::BYTES + WAVES * 16 * TQ) + wave * CAND;   // [CAND] score bits; column | vector of the part << 7 | place among the column's << 19
    float* s_g = reinterpret_cast<float*>(table + Tab::BYTES + WAVES * (16 * TQ + 8 * CAND)) + wave * 64;         // [32] 2^-20 * norms of the slab, ...
    float* s_x = s_g + 32;                                                                       // [32] ... and its vectors' lengths (RAW)
    int* s_cnt = reinterpret_cast<int*>(table + Tab::BYTES + WAVES * (16 * TQ + 8 * CAND + 64 * 4)) + wave * (TQ + 2);     // [TQ] held back per column, then their first position
    int* s_held = s_cnt + TQ;                                                                    // [2] asked for, held back if that is too many
    constexpr float kUnscale = 1.f / (kSplitScale * kSplitScale);

    Tab::fill(table, a.cb, 64 * WAVES);
    const uint32_t own = (uint32_t)(tid % Tab::TC * Tab::ENTRY);
    const int words = a.store.words;
    const SlabWords<DP, B, NW> from{words, half, jl};
    for (int e = lane; e < TQ; e += 64) s_cnt[e] = 0;
    if (lane == 0) { s_held[0] = 0; s_held[1] = CAND; }
    __syncthreads();
    for (TileQueue<TQ> queue(a, wave, WAVES); queue.tile < queue.end; queue.advance()) {
    const BatchTile t = queue.t;
    const int n_v = t.v_hi - t.v_lo, nslab = (n_v + 31) / 32, n_qt = (t.nq_tile + 31) / 32;
    // A list starts at a multiple of 64 slots and its slots reach to one, so a slab's words and norms can be read whole; the norms of
    // what lies beyond the list count as no numbers.
    const int64_t slot0 = t.base_slot + t.v_lo;
    const uint32_t* codes = a.store.codes + (slot0 >> 6) * words * 64;
    auto slab_at = [&](int slab) { return codes + (int64_t)(slab >> 1) * words * 64 + (slab & 1) * 32; };

    auto scan = [&](auto tiles) {
        constexpr int N = decltype(tiles)::value;
        // Words and norm of a slab on their way: two slabs ahead of the products, or one where the registers do not reach for two.
        constexpr int AHEAD = 4 * KB * N + 16 * N + 2 * KB * NW <= 200 ? 2 : 1;
        struct Ahead { uint32_t w[KB][NW], g16; float xn; } ahead[AHEAD];
        auto fetch_norm = [&](int slab, Ahead& f) {
            f.g16 = (a.store.gamma + slot0 + slab * 32)[lane_offset(jl)];
            if (RAW) f.xn = (a.store.xnorm + slot0 + slab * 32)[lane_offset(jl)];
        };
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) {
            const int slab = i < nslab ? i : 0;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) from.load(slab_at(slab), kb, ahead[i].w[kb]);
            fetch_norm(slab, ahead[i]);
        }
        half8 qh[N][KB];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const int e = 32 * n + jl;
            const int32_t it = queue.pair_of(e), q = it / a.np;
            load_query<DP>(a.zh + (int64_t)q * a.z_pitch + 8 * half, a.z_pitch, qh[n]);
            // (columns beyond the tile's queries: a NaN threshold, which not even an infinite score reaches; both halves write the same)
            s_row[e] = make_uint4(__float_as_uint(a.coarse[it]), e < t.nq_tile ? __float_as_uint(a.thresh[(int64_t)q * a.thresh_stride]) : 0x7FC00000u,
                                  (uint32_t)it, RAW ? __float_as_uint(a.qnorm[q]) : 0u);
        }
        queue.proceed();
        wave_sync();
        auto scan_slab = [&](int slab, Ahead& f) {
            // A block's words make room for those of the same block AHEAD slabs on as soon as they are looked up.
            const int next = slab + AHEAD < nslab ? slab + AHEAD : slab;
            const uint32_t* next_at = slab_at(next);
            constexpr int EARLY = N < 3 ? 2 : 1;         // blocks in flight ahead of the products
            typename Tab::Raw raw[EARLY + 1];
            auto look = [&](int kb) {
                Tab::look_up(table, own, code_chunk<B, NW>(f.w[kb], kb, half), raw[kb % (EARLY + 1)]);
                from.load(next_at, kb, f.w[kb]);
            };
#pragma unroll
            for (int kb = 0; kb < EARLY && kb < KB; ++kb) look(kb);
            // 2^-20 * norm of vector jl; the largest of the slab (numbers that are not negative have the order of their bits), for a raw
            // metric also the range of the vectors' lengths.  A length that is no number makes its own score none and leaves the range as
            // it is: as the slab's largest it would hide the others'.
            const bool in_part = slab * 32 + jl < n_v;
            const float g_own = in_part ? kUnscale * __half2float(__ushort_as_half((uint16_t)f.g16)) : __builtin_nanf("");
            s_g[jl] = g_own;
            const float g_max = __int_as_float(slab_max(g_own == g_own ? __float_as_int(g_own) : 0));
            float x_min = 0.f, x_max = 0.f;
            if (RAW) {
                s_x[jl] = f.xn;
                const bool counts = in_part && f.xn == f.xn;
                x_min = __int_as_float(~slab_max(counts ? ~__float_as_int(f.xn) : INT32_MIN));
                x_max = __int_as_float(slab_max(counts ? __float_as_int(f.xn) : 0));
            }
            fetch_norm(next, f);
            wave_sync();
            floatx16 acc[N];
#pragma unroll
            for (int n = 0; n < N; ++n)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[n][r] = 0.f;
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                if (kb + EARLY < KB) look(kb + EARLY);
                half8 vh, none;
                Tab::operands(raw[kb % (EARLY + 1)], vh, none);
#pragma unroll
                for (int n = 0; n < N; ++n) acc[n] = __builtin_amdgcn_mfma_f32_32x32x16_f16(vh, qh[n][kb], acc[n], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            // No row of a tile can reach the threshold unless the largest accumulator times the largest norm
            // does: g_max >= g_r >= 0 and a_max >= max(acc_r, 0), and a correctly rounded sum or fused multiply-add never
            // decreases when its exact value grows, so fmaf(g_max, a_max + acc0, sq) >= fmaf(g_r, acc_r + acc0, sq).
#pragma unroll
            for (int n = 0; n < N; ++n) {
                const int e = 32 * n + jl;
                const uint2 row = *reinterpret_cast<const uint2*>(s_row + e);
                const float sq = __uint_as_float(row.x), th = __uint_as_float(row.y);
                float a_max = 0.f;
#pragma unroll
                for (int r = 0; r < 16; r += 2) a_max = fmaxf(fmaxf(a_max, acc[n][r]), acc[n][r + 1]);
                float top = fmaf(g_max, a_max + a.acc0, sq);
                if (RAW) top = metric_key_bound(a.metric, top, x_min, x_max, __uint_as_float(s_row[e].w));
                if (!(top >= th)) continue;        // seldom: some row of this lane may reach the threshold
                const float qn = RAW ? __uint_as_float(s_row[e].w) : 0.f;
                // The keys take the place of the sums.  Counted first: one update of the query's counter for all of the lane's rows (its
                // latency, once per row, was 2/3 of the pass where 1 in 80 vectors is appended).
                int v0 = 4 * half;
                asm volatile("" : "+v"(v0));       // (or every row's address is prepared ahead of the tiles and spilled)
                uint32_t hit = 0;
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int at = v0 + 8 * (r / 4) + (r % 4);
                    float u = fmaf(s_g[at], acc[n][r] + a.acc0, sq);  // upper bound of the score; NaN never passes
                    if (RAW) u = metric_key(a.metric, u, s_x[at], qn);
                    acc[n][r] = u;
                    hit |= u >= th ? 1u << r : 0u;
                }
                if (!hit) continue;
                const int n_hit = (int)__popc(hit), v1 = slab * 32 + v0;      // v1: number of the lane's first row in the part
                int held = atomicAdd(&s_held[0], n_hit);
                if (held + n_hit <= CAND) {
                    uint32_t word = (uint32_t)(e | v1 << 7) + ((uint32_t)atomicAdd(&s_cnt[e], n_hit) << 19);
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if ((hit >> r) & 1u) {
                            s_cand[held++] = make_uint2(__float_as_uint(acc[n][r]), word + ((uint32_t)(8 * (r / 4) + (r % 4)) << 7));
                            word += 1u << 19;
                        }
                } else {
                    atomicMin(&s_held[1], held);
                    const int32_t it = (int32_t)s_row[e].z, q = it / a.np;
                    const int64_t rank = (int64_t)(it - q * a.np) << kCandProbeShift;
                    const int pos = atomicAdd(&a.cand_cnt[q], n_hit);
                    const int room = a.cap - pos;
                    float* to_score = a.cand_score + (int64_t)q * a.cap + pos;
                    int64_t* to_slot = a.cand_slot + (int64_t)q * a.cap + pos;
                    const int64_t first = (slot0 + v1) | rank;       // adding to the slot stays below the rank
                    int at = 0;
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if ((hit >> r) & 1u) {
                            if (at < room) {
                                to_score[at] = acc[n][r];
                                to_slot[at] = first + 8 * (r / 4) + (r % 4);
                            }
                            ++at;
                        }
                }
            }
        };
        for (int slab = 0; slab < nslab; slab += AHEAD) {
            scan_slab(slab, ahead[0]);
            if (AHEAD > 1 && slab + 1 < nslab) scan_slab(slab + 1, ahead[AHEAD - 1]);
            queue.between(slab);
        }
    };
    if (NQ >= 4 && n_qt == 4) scan(std::integral_constant<int, NQ >= 4 ? 4 : 1>{});
    else if (NQ >= 3 && n_qt == 3) scan(std::integral_constant<int, NQ >= 3 ? 3 : 1>{});
    else if (n_qt == 2) scan(std::integral_constant<int, 2>{});
    else scan(std::integral_constant<int, 1>{});

    wave_sync();
    const int asked = __builtin_amdgcn_readfirstlane(s_held[0]);
    if (asked > 0) {                             // what this tile held back
        const int held = asked <= CAND ? asked : __builtin_amdgcn_readfirstlane(s_held[1]);      // (once one did not fit, none after it did)
        for (int e = lane; e < TQ; e += 64)
            if (s_cnt[e] > 0) s_cnt[e] = atomicAdd(&a.cand_cnt[(int32_t)s_row[e].z / a.np], s_cnt[e]);
        wave_sync();
        for (int i = lane; i < held; i += 64) {
            const uint2 c = s_cand[i];
            const int e = (int)(c.y & 127u);
            const int32_t it = (int32_t)s_row[e].z, q = it / a.np;
            const int pos = s_cnt[e] + (int)(c.y >> 19);
            if (pos < a.cap) {
                a.cand_score[(int64_t)q * a.cap + pos] = __uint_as_float(c.x);
                a.cand_slot[(int64_t)q * a.cap + pos] = (slot0 + (int)((c.y >> 7) & 4095u)) | (int64_t)(it - q * a.np) << kCandProbeShift;
            }
        }
        wave_sync();
        for (int e = lane; e < TQ; e += 64) s_cnt[e] = 0;
        if (lane == 0) { s_held[0] = 0; s_held[1] = CAND; }
        wave_sync();
    }
    }
}

template <int DP, int B>
struct BatchForm {
    static constexpr int NQ = batch_query_tiles(DP, B);
    static constexpr int OCC = 2;
    static_assert(32 * NQ >= kBatchTile, "the room for tiles is counted by the fewest queries of one");
    static_assert(32 * NQ <= kBatchTileMost, "and which calls have few of them by the most");
};

template <int DP, int B>
hipError_t run_batch(const BatchScanArgs& a, hipStream_t st) {
    using Form = BatchForm<DP, B>;
    static ChipFill fill[4];
    const auto go = [&](ChipFill& own, auto kernel, int occ, size_t lds) -> hipError_t {
        unsigned wgs = 0;
        const hipError_t e = own.get(reinterpret_cast<const void*>(kernel), 64 * waves_of(occ), lds, &wgs);
        if (e == hipSuccess) hipLaunchKernelGGL(kernel, dim3((unsigned)tile_workgroups((int)wgs)), dim3(64 * waves_of(occ)), lds, st, a);
        return e;
    };
    constexpr int OCC = Form::OCC, NQ = Form::NQ;
    constexpr size_t lds_near = Table<B, true>::BYTES, lds = ThresholdCfg<DP, B, NQ, OCC>::lds;
    const hipError_t e = a.dense    ? a.metric ? go(fill[0], k_batch_dense<DP, B, true>, DenseCfg<DP, B, true>::OCC, lds_near)
                                               : go(fill[1], k_batch_dense<DP, B, false>, DenseCfg<DP, B, false>::OCC, lds_near)
                         : a.metric ? go(fill[2], k_batch_threshold<DP, B, NQ, OCC, true>, OCC, lds)
                                    : go(fill[3], k_batch_threshold<DP, B, NQ, OCC, false>, OCC, lds);
    return e != hipSuccess ? e : hipGetLastError();
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
