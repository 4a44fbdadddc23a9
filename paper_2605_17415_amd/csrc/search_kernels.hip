// Search-side kernels (Section "Architecture", Search): the scan of the probed lists, which adds
// the residual estimate gamma * <Pi q~, C[code]> to the exact coarse term, and the per-query
// selection of the best k (also used to pick the nprobe best cells).
#include <hip/hip_fp16.h>

#include <algorithm>

#include "kernels.h"
#include "wave_sum.h"

namespace ivftq {

namespace {

// ---- candidate offsets -----------------------------------------------------------------------

// inclusive sum of v over the wavefront's lanes
__device__ __forceinline__ int32_t lanes_up_to(int32_t v, int lane) {
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}

// The place of pair (q, p) of cell `list` in its bucket: the query's nearest p1 lists in one, the others in another.
__device__ __forceinline__ void count_pair(const CandOffsetArgs& c, int64_t q, int np, int p, int p1, int list) {
    if (c.rank && p < np && list >= 0) c.rank[q * np + p] = (int32_t)atomicAdd(&c.bucket_cnt[list + (p >= p1 ? c.L : 0)], 1u);
}

// How many of a query's `total` candidates are scored densely to find its threshold.  Were the prefix a random
// sample of P of the query's T candidates, its k-th score would be beaten by about k*(T-P)/P of the others;
// P = f*k*T/cap (f = kPrefixFactorX2/2) keeps that near cap/f even then.  The nearest lists hold the best
// candidates, so in practice far fewer pass (and a list that does overflow sends its query to the exact pass).  At
// least k vectors, so that a threshold exists.
__device__ __forceinline__ int64_t dense_prefix(const CandOffsetArgs& c, int32_t total) {
    const int64_t need = (kPrefixFactorX2 * (int64_t)c.k * total + 2 * c.cap - 1) / (2 * c.cap);
    return need < c.k ? c.k : need;
}

// one lane: the prefix of query q, and its counters of the batched scan (cleared here rather than by launches of their own)
__device__ __forceinline__ void put_first(const CandOffsetArgs& c, int64_t q, int p1) {
    c.first[q] = p1;
    if (c.cand_cnt) c.cand_cnt[q] = 0;
    if (c.redo_cnt) c.redo_cnt[q] = c.redo_done[q] = 0;
    if (c.gate && q == 0) c.gate[0] = 0;
}

// The same for the probes of a query held by the lanes of a wavefront (np <= 64; `list` is ignored beyond np).
__device__ __forceinline__ void cand_offsets_lanes(const CandOffsetArgs& c, int64_t q, int np, int list, int lane) {
    const int32_t size = lane < np && list >= 0 ? c.list_size[list] : 0;
    const int32_t incl = lanes_up_to(size, lane);
    const int32_t total = __shfl(incl, 63);
    int32_t* off = c.cand_off + q * (np + 1);
    if (lane < np) off[lane] = incl - size;
    if (lane == 0) off[np] = total;
    if (!c.first) return;
    const uint64_t reached = __ballot(lane < np && (int64_t)incl >= dense_prefix(c, total));
    const int p1 = reached ? (int)__builtin_ctzll(reached) + 1 : np;
    count_pair(c, q, np, lane, p1, list);
    if (lane == 0) put_first(c, q, p1);
}

// And for any number of probes, whose cells are in LDS: 64 at a time, `incl` ([np], LDS) takes the running sums.
__device__ __forceinline__ void cand_offsets_wave(const CandOffsetArgs& c, int64_t q, int np, const int32_t* cell, int32_t* incl, int lane) {
    int32_t* off = c.cand_off + q * (np + 1);
    int32_t run = 0;
    for (int p0 = 0; p0 < np; p0 += 64) {
        const int p = p0 + lane, list = p < np ? cell[p] : -1;
        const int32_t size = list >= 0 ? c.list_size[list] : 0;
        const int32_t upto = run + lanes_up_to(size, lane);
        if (p < np) { off[p] = upto - size; incl[p] = upto; }
        run = __shfl(upto, 63);
    }
    if (lane == 0) off[np] = run;
    if (!c.first) return;
    // the first p >= 1 whose lists 0 .. p-1 together reach `need` (np when none does); a lane reads what it wrote
    const int64_t need = dense_prefix(c, run);
    int p1 = np;
    for (int p0 = 0; p0 < np && p1 == np; p0 += 64) {
        const uint64_t reached = __ballot(p0 + lane < np && (int64_t)incl[p0 + lane] >= need);
        if (reached) p1 = p0 + (int)__builtin_ctzll(reached) + 1;
    }
    for (int p = lane; p < np; p += 64) count_pair(c, q, np, p, p1, cell[p]);
    if (lane == 0) put_first(c, q, p1);
}

// Order-preserving key of a score; whatever is no number gets 0, which no score has: it is no cell and no result.
__device__ __forceinline__ uint32_t order_key(float f) {
    const uint32_t u = __float_as_uint(f);
    return f != f ? 0u : u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);      // (all bits of a negative one, the sign of another)
}
__device__ __forceinline__ float order_value(uint32_t key) { return __uint_as_float((key & 0x80000000u) ? (key ^ 0x80000000u) : ~key); }

// ---- the k best of a query redone exactly ---------------------------------------------------------
//
// By one workgroup, from redo_cnt[q] scores in arbitrary order at `vals` and the candidate columns
// they belong to.  An entry's composite (order-preserving key of the score, then ~column) makes all entries
// distinct: the k with the largest composites are the k best, ties going to the smaller column, whatever the
// order they were appended in.  A radix search narrows the entries down, a byte at a time, until at most
// max(k, kRedoFew) reach what is known of the k-th largest composite; those are gathered and sorted in LDS.  Bound by
// the latency of its passes and of the sort's barriers; on the benchmark's searches one to three queries of 10,000
// come here, with 400 to 3000 entries each.  Sorting up to 2048 entries outright, and all eight passes beyond, with the
// digit looked for by one thread, took 50 us at 10M x 96 (k = 10); 13 us with the radix search.
constexpr int kRedoSort = 2048, kRedoFew = 128;
static_assert(kMaxK <= kRedoSort, "the k winners are sorted in LDS");
constexpr size_t kRedoLds = kRedoSort * 16 + 256 * 4 + 16;

template <int NT>
__device__ __forceinline__ void redo_select(const ListScanArgs& a, int64_t q, const float* vals, unsigned char* lds) {
    uint64_t* s_comp = reinterpret_cast<uint64_t*>(lds);              // [kRedoSort]
    int64_t* s_lab = reinterpret_cast<int64_t*>(s_comp + kRedoSort);  // [kRedoSort]
    uint32_t* hist = reinterpret_cast<uint32_t*>(s_lab + kRedoSort);  // [256]
    uint32_t* ctrl = hist + 256;                                      // [3]
    const int tid = threadIdx.x;
    const int32_t* off = a.cand_off + q * (a.np + 1);
    const int n = __hip_atomic_load(&a.redo_cnt[q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const float* cols = vals + a.m_stride / 2;
    auto comp_of = [&](int i) -> uint64_t {
        return ((uint64_t)order_key(vals[i]) << 32) | (uint32_t)~__float_as_uint(cols[i]);
    };
    const int take = n < a.k ? n : a.k;
    uint64_t last = 0;                          // every entry of at least this composite is gathered
    const int few = take > kRedoFew ? take : kRedoFew;
    if (n > few) {
        uint64_t mask = 0;
        uint32_t need = (uint32_t)take;             // winners among the entries that share the bytes found so far
        for (int shift = 56; shift >= 0; shift -= 8) {
            __syncthreads();
            if (tid < 256) hist[tid] = 0;
            __syncthreads();
            for (int i = tid; i < n; i += NT) {
                const uint64_t c = comp_of(i);
                if ((c & mask) == last) atomicAdd(&hist[(c >> shift) & 255u], 1u);
            }
            __syncthreads();
            if (tid < 64) {                         // the digit where the running count, from above, first reaches `need`
                uint32_t h[4];                      // lane l owns digits 4l .. 4l+3
#pragma unroll
                for (int e = 0; e < 4; ++e) h[e] = hist[4 * tid + e];
                const uint32_t own = h[0] + h[1] + h[2] + h[3];
                uint32_t above = own;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t t = __shfl_down(above, o);
                    if (tid + o < 64) above += t;
                }
                above -= own;
#pragma unroll
                for (int e = 3; e >= 0; --e) {
                    if (above < need && above + h[e] >= need) {         // true for one digit only
                        ctrl[0] = (uint32_t)(4 * tid + e);
                        ctrl[1] = need - above;
                        ctrl[2] = h[e];
                    }
                    above += h[e];
                }
            }
            __syncthreads();
            last |= (uint64_t)ctrl[0] << shift;
            mask |= (uint64_t)255 << shift;
            need = ctrl[1];
            // (all that reach `last`: the winners beyond its bytes, and every entry that shares them)
            if ((uint32_t)take - need + ctrl[2] <= (uint32_t)few) break;
        }
    }
    __syncthreads();
    if (tid == 0) ctrl[0] = 0;
    __syncthreads();
    for (int i = tid; i < n; i += NT) {
        const uint64_t c = comp_of(i);
        if (c >= last) {
            const uint32_t at = atomicAdd(&ctrl[0], 1u);
            if (at < (uint32_t)kRedoSort) s_comp[at] = c;
        }
    }
    __syncthreads();
    const int got = min((int)ctrl[0], kRedoSort);
    int size = 1;
    while (size < got) size <<= 1;
    for (int i = got + tid; i < size; i += NT) s_comp[i] = 0;
    __syncthreads();
    for (int sz = 2; sz <= size; sz <<= 1)
        for (int stride = sz >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < size / 2; i += NT) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const uint64_t c0 = s_comp[lo], c1 = s_comp[hi];
                if ((c0 >= c1) != ((lo & sz) == 0)) { s_comp[lo] = c1; s_comp[hi] = c0; }
            }
            __syncthreads();
        }
    // labels of the winners, then equal scores in label order
    int kpad = 1;
    while (kpad < take) kpad <<= 1;
    for (int i = tid; i < kpad; i += NT) {
        int64_t lab = INT64_MAX;
        if (i < take) {
            const int32_t col = (int32_t)~(uint32_t)s_comp[i];
            int lo = 0, hi = a.np;              // largest p with off[p] <= col
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (off[mid] <= col) lo = mid; else hi = mid;
            }
            const int64_t slot = a.store.list_off[a.probe[q * a.np + lo]] + (col - off[lo]);
            lab = a.ids ? a.ids[slot] : slot;
        } else {
            s_comp[i] = 0;
        }
        s_lab[i] = lab;
    }
    __syncthreads();
    for (int sz = 2; sz <= kpad; sz <<= 1)
        for (int stride = sz >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < kpad / 2; i += NT) {
                const int lo = 2 * i - (i & (stride - 1)), hi = lo + stride;
                const uint32_t k0 = (uint32_t)(s_comp[lo] >> 32), k1 = (uint32_t)(s_comp[hi] >> 32);
                const int64_t l0 = s_lab[lo], l1 = s_lab[hi];
                if ((k0 > k1 || (k0 == k1 && l0 <= l1)) != ((lo & sz) == 0)) {
                    const uint64_t c = s_comp[lo]; s_comp[lo] = s_comp[hi]; s_comp[hi] = c;
                    s_lab[lo] = l1; s_lab[hi] = l0;
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < a.k; i += NT) {
        const uint32_t key = i < take ? (uint32_t)(s_comp[i] >> 32) : 0u;
        const float v = i < take ? order_value(key) : -__builtin_inff();
        a.out_vals[q * a.k + i] = a.metric ? metric_value(a.metric, v, a.qnorm[q]) : v;
        a.out_i64[q * a.k + i] = i < take ? s_lab[i] : -1;
    }
}

// ---- list scan: a row of workgroups per query walks its probed lists ---------------------------
//
// The query's rotated coordinates and the 2^b centroid values are combined once per workgroup
// into a table lut[j][e] = z_j * C[e] in LDS (the per-query ADC table the paper's own scan uses,
// Appendix "Why cascade does not yield a speedup"); a lane then owns one stored vector at a time,
// reads its packed words with 256-byte-per-wavefront coalesced loads and sums d table entries.
// When the table would not fit LDS (large b and d) DIRECT keeps z and C separately and multiplies
// per coordinate instead.
//
// REDO: only the queries that overflowed their candidate list (launch_list_scan), and only scores that reach the
// query's threshold are kept, with their columns, in arbitrary order.  A launch mostly finds no such query or a
// few, so all of its workgroups are shared out over those it finds: two queries of 64 lists on eight workgroups
// each took 0.66 ms at 10M x 200, each workgroup walking eight lists alone; spread over the chip 0.02 ms.  The last workgroup to
// finish its share of a query selects its results.  When there are more such queries than workgroups, every workgroup takes queries by itself, one
// after the other in a row of its own.  (Full-length rows are few, 1500 for 10,000 queries x 64 probes of 10M x 200; with a scan and a
// selection for every turn of them, most of them empty, the redo of a query or none took 64 us there, and 56 for 32 probes of 10M x 96;
// one launch takes 28, or 4 when it finds nothing.)  Workgroups are small and few enough in registers that the chip holds all of them at once:
// with half as many of 1024 threads, 71 registers a lane and so one to a compute unit, a query of many was selected while others waited for
// a place (4000 queries x 32 probes, 400,000 x 16, 176 of them redone: 147 us, now 81; two launches took 79).
//
// redo_margin: how far a score s_l + g * sum can lie below its evaluation by the dense pass, from which the threshold
// comes.  slack bounds the difference of the two sums; it counts for every unit of the norm, which a caller's own
// codes may have at any size, and the sum with the coarse term is rounded at the size of that.
__device__ __forceinline__ float redo_margin(float slack, float s_l, float g) { return slack * fmaxf(g, 1.f) + 0x1p-21f * fabsf(s_l); }

// BLK: every block of 64 vectors of a list leaves the key of its best score beside the scores, so that the
// selection reads a 64th of the row and then the few blocks that can hold a result (block_index).  A form of its own: tested at run
// time, and with lanes past a list's end kept for the exchange, lists of few vectors took up to 15 % longer (3008 queries x 44 lists of 4
// 91 us instead of 79, 5461 x 54 of 17 252 instead of 232).
template <int B, bool DIRECT, bool REDO, bool BLK>
__global__ __launch_bounds__(REDO ? kRedoThreads : 256) __attribute__((amdgpu_waves_per_eu(!REDO ? 1 : B <= 4 || DIRECT ? 8 : B <= 6 ? 6 : 5, 8))) void k_list_scan(ListScanArgs a) {
    constexpr int K = 1 << B, NT = REDO ? kRedoThreads : 256;
    extern __shared__ float lut[];     // [d][K], or z[d] followed by C[K] when DIRECT
    const float* __restrict__ z = a.z;
    const float* __restrict__ cb = a.cb;
    const int32_t* __restrict__ probe = a.probe;
    const float* __restrict__ coarse = a.coarse;
    const int32_t* __restrict__ cand_off = a.cand_off;
    const ListStore& store = a.store;
    const int z_pitch = a.z_pitch, d = a.d, np = a.np, metric = a.metric;
    // this workgroup takes the probes p_first, p_first + p_step, ... of a query and of each of those lists the
    // rounds slice, slice + slices, ... of 256 vectors
    int64_t row = blockIdx.y, row_step = 1, row_end = row + 1;
    int p_first = (int)blockIdx.x, p_step = (int)gridDim.x, slice = (int)blockIdx.z, slices = (int)gridDim.z;
    int64_t buffer = row;              // score row
    if constexpr (REDO) {
        const int n_redo = min(a.gate[0] - a.gate_begin, a.gate_count);
        if (n_redo <= 0) return;
        const int per = min(512, max(1, (int)gridDim.x / n_redo));       // workgroups per query (each costs its counter 14 ns)
        const int part = (int)blockIdx.x % per;
        row = buffer = (int)blockIdx.x / per; row_step = (int)gridDim.x / per; row_end = n_redo;
        if (row >= row_step) return;
        p_step = min(per, np);
        slices = per / p_step;
        p_first = part % p_step;
        slice = part / p_step;
        if (slice >= slices) return;
    }
    for (; row < row_end; row += row_step) {
    if constexpr (!REDO) buffer = row;
    const int64_t q = REDO ? a.gate[1 + a.gate_begin + row] : row;
    if (p_first >= np) continue;
    const float qn = metric ? a.qnorm[q] : 1.f;
    float reach = 0.f;
    if constexpr (REDO) {
        reach = a.thresh[q * a.thresh_stride];
        __syncthreads();               // the table of the previous query is no longer read
    }

    if constexpr (DIRECT) {
        for (int e = threadIdx.x; e < d; e += NT) lut[e] = z[q * z_pitch + e];
        for (int e = threadIdx.x; e < K; e += NT) lut[d + e] = cb[e];
    } else {
        for (int e = threadIdx.x; e < d * K; e += NT) lut[e] = z[q * z_pitch + (e >> B)] * cb[e & (K - 1)];
    }
    __syncthreads();
    auto term = [&](int j, uint32_t code) -> float {
        if constexpr (DIRECT) return lut[j] * lut[d + code];
        else return lut[j * K + code];
    };

    const int words = store.words;
    for (int p = p_first; p < np; p += p_step) {
    const int l = probe[q * np + p], cell = l < 0 ? 0 : l;
    const int size = store.list_size[cell], n_l = l < 0 ? 0 : size;     // (no cell: a query whose scores are no numbers)
    const float s_l = coarse[q * np + p];
    const int64_t base_slot = store.list_off[cell];
    const int32_t col0 = cand_off[q * (np + 1) + p];
    float* out = a.scores + buffer * a.m_stride + (REDO ? 0 : col0);
    const int lane = (int)(threadIdx.x & 63);
    uint32_t* blk = nullptr;
    if constexpr (BLK) {
        blk = a.blk_max + row * a.blk_stride + block_index(col0, p);
        // places between this list's blocks and the next one's hold nothing
        const int own = block_index(cand_off[q * (np + 1) + p + 1], p + 1) - block_index(col0, p);
        const int b = (n_l + 63) / 64 + (int)threadIdx.x;
        if (slice == 0 && b < own) blk[b] = 0u;
    }

    // a list is dealt out in rounds of a vector per thread to the workgroups that share it
    for (int v0 = NT * slice + (int)(threadIdx.x & ~63u); v0 < n_l; v0 += NT * slices) {
        const int v = v0 + lane;
        const bool in_list = v < n_l;
        if (!REDO && !BLK && !in_list) break;
        const int64_t slot = base_slot + (in_list ? v : n_l - 1);
        const uint32_t* wp = store.codes + (slot >> 6) * words * 64 + (slot & 63);
        float acc = 0.f;
        // A row is walked in chunks of 32 coordinates = B packed words, whose codes sit at bit positions known at
        // compile time.
        int chunks = 0;                // whole chunks summed by the table lookups below
        if constexpr (!DIRECT && B >= 2) {   // (one-bit codes: the two bits below a code are not a single neighbour's)
            // Table lookups without address arithmetic.  The codes of a word are split by the parity of their
            // position into two masked copies, so that the bits below a code are zero; a bit-field extract that
            // starts two bits below the code then yields the code times four, the byte offset of its table entry.
            // The chunk loop is unrolled against the longest row the table fits, which makes the coordinate's part
            // of the address an immediate of the LDS read: per code one extract, one read and one add, per word
            // two masks.  (A code in the lowest two bits of a word is shifted up and masked instead, one that
            // straddles two words is taken from the aligned pair.)  The next chunk's words are fetched before the
            // current one is summed.  Coordinates beyond the last whole chunk take the loop further down.
            // longest row: the table fits 64 KB (4K bytes per coordinate) and the library takes d <= 256
            constexpr int kMaxCoords = (64 * 1024 / (K * 4)) < 256 ? (64 * 1024 / (K * 4)) : 256;
            constexpr int kMaxChunks = kMaxCoords / 32;
            // The table's LDS address: the lookups address LDS by number (offset of the entry plus an
            // immediate), which holds when the table starts at LDS address 0 -- it is this kernel's only
            // shared array; were it ever placed elsewhere, every chunk takes the loop further down instead.
            typedef __attribute__((address_space(3))) const float lds_float;
            uint32_t lut_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)lut;
            asm volatile("" : "+s"(lut_at));
            // opaque, so that the tests below stay scalar compares inside the loop instead of a set of flags
            // computed ahead of it
            chunks = lut_at == 0 ? ((d >> 5) < kMaxChunks ? (d >> 5) : kMaxChunks) : 0;
            asm volatile("" : "+s"(chunks));
            uint32_t cur[B];
            if (chunks > 0) {
#pragma unroll
                for (int u = 0; u < B; ++u) cur[u] = wp[u * 64];
            }
#pragma unroll
            for (int c = 0; c < kMaxChunks; ++c) {
                if (c >= chunks) break;
                uint32_t nxt[B];
                if (c + 1 < chunks) {
#pragma unroll
                    for (int u = 0; u < B; ++u) nxt[u] = wp[((c + 1) * B + u) * 64];
                }
                uint32_t par[B][2];    // word u with only its whole codes of even / odd position kept
#pragma unroll
                for (int u = 0; u < B; ++u) {
                    uint32_t m[2] = {0u, 0u};
#pragma unroll
                    for (int t = 0; t < 32; ++t)
                        if (((t * B) >> 5) == u && ((t * B) & 31) + B <= 32) m[t & 1] |= (uint32_t)(K - 1) << ((t * B) & 31);
                    par[u][0] = cur[u] & m[0];
                    par[u][1] = cur[u] & m[1];
                    asm("" : "+v"(par[u][0]));   // keeps each lookup one bit-field extract: with the cleared
                    asm("" : "+v"(par[u][1]));   // bits known, the compiler rewrites it as a shift and a mask
                }
#pragma unroll
                for (int t = 0; t < 32; ++t) {
                    const int wi = (t * B) >> 5, sh = (t * B) & 31;
                    uint32_t off4;
                    if (sh + B > 32)   // straddles: sh > 24
                        off4 = __builtin_amdgcn_alignbit(cur[wi + 1 < B ? wi + 1 : wi], cur[wi], sh - 2) & ((uint32_t)(K - 1) << 2);
                    else if (sh < 2)
                        off4 = (cur[wi] << (2 - sh)) & ((uint32_t)(K - 1) << 2);
                    else
                        off4 = __builtin_amdgcn_ubfe(par[wi][t & 1], sh - 2, B + 2);
                    acc += *(lds_float*)(off4 + (uint32_t)((c * 32 + t) * K * 4));
                }
#pragma unroll
                for (int u = 0; u < B; ++u) cur[u] = nxt[u];
            }
        }
        // the rest (a last chunk of fewer than 32 coordinates; every chunk when the table is not in LDS): every
        // code is one bit-field extract (two shifts where it straddles a word) plus the address arithmetic
        for (int w0 = chunks * B; w0 < words; w0 += B) {
            uint32_t wd[B + 1];
#pragma unroll
            for (int u = 0; u < B; ++u) wd[u] = (w0 + u < words) ? wp[(w0 + u) * 64] : 0u;
            wd[B] = 0u;
            const int j0 = (w0 / B) * 32;
            const bool whole = j0 + 32 <= d;
#pragma unroll
            for (int t = 0; t < 32; ++t) {
                constexpr int kBits = B;
                const int wi = (t * kBits) >> 5, sh = (t * kBits) & 31;
                const uint32_t code = (sh + kBits <= 32)
                    ? __builtin_amdgcn_ubfe(wd[wi], sh, kBits)
                    : (((wd[wi] >> sh) | (wd[wi + 1] << (32 - sh))) & (uint32_t)(K - 1));
                if (whole || j0 + t < d) acc += term(j0 + t, code);
            }
        }
        const float g = __half2float(__ushort_as_half(store.gamma[slot]));
        float sc = s_l + g * acc;
        float margin = 0.f;
        if (metric) {                  // ranking key of a raw metric (metric_value turns the selected ones into values)
            const float xn = store.xnorm[slot];
            if constexpr (REDO) margin = fabsf(metric_scale(metric, xn, qn)) * redo_margin(a.slack, s_l, g);
            sc = metric_key(metric, sc, xn, qn);
            if constexpr (REDO) margin += 0x1p-21f * fabsf(sc);
        } else if constexpr (REDO) {
            margin = redo_margin(a.slack, s_l, g);
        }
        if constexpr (REDO) {
            const bool keep = in_list && sc == sc && !(sc < reach - margin);     // (a margin that is no number keeps what is one)
            const uint64_t in = __ballot(keep);           // one counter update per wavefront
            if (in) {
                const int leader = (int)__builtin_ctzll(in);
                int at = 0;
                if (lane == leader) at = atomicAdd(&a.redo_cnt[q], (int)__popcll(in));
                at = __shfl(at, leader) + (int)__popcll(in & (((uint64_t)1 << lane) - 1));
                if (keep) {
                    __hip_atomic_store(out + at, sc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    __hip_atomic_store(out + a.m_stride / 2 + at, __int_as_float(col0 + v), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        } else {
            if (in_list) out[v] = sc;
            if constexpr (BLK) {
                uint32_t key = in_list ? order_key(sc) : 0u;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) key = max(key, (uint32_t)__shfl_xor(key, o));
                if (lane == 0) blk[v0 >> 6] = key;
            }
        }
    }
    }
    if constexpr (REDO) {
        // What every workgroup kept has to be there for the one that comes last, maybe on another part of the chip with an L2 cache
        // of its own.  The language orders that by a release alone, which here means writing the L2 cache back, although nothing of this
        // lies in it: stores of agent scope go through it to memory, and a wavefront's wait ends when its own are there.  So each wavefront
        // waits for its stores, in a statement that the compiler moves no store across, the workgroup meets, and one thread counts for
        // it.  That holds for gfx950, which this is written for.  (A fence by every wavefront: 160 us a redo; a release by the counting
        // thread alone: 37 instead of 28.5 for few queries at 10M x 96, the call 3 % slower, 93 instead of 82 for 176 of 4000.)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        unsigned char* lds = reinterpret_cast<unsigned char*>(lut);
        int* s_last = reinterpret_cast<int*>(lds + kRedoLds) - 1;         // (behind the selection's three control words)
        if (threadIdx.x == 0) *s_last = atomicAdd(&a.redo_done[q], 1) == p_step * slices - 1;
        __syncthreads();
        if (*s_last != 0) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __syncthreads();
            redo_select<NT>(a, q, a.scores + buffer * a.m_stride, lds);
        }
    }
    }
}

// ---- selection: k largest of a row ------------------------------------------------------------
//
// One workgroup per row, exact, on an order-preserving 32-bit key.  Keys equal to the k-th largest are kept in column
// order; the winners are labelled and ordered by (value desc, label asc).
//
// Short cut (up to kSelTake winners).  The row is split into parts, of which the largest keys are known: the parts are the
// blocks of 64 columns whose maxima the scan left (blk_max), or the columns dealt out round-robin to the 256 threads.
// Every thread holds the largest of its share of these maxima; at least `take` keys reach the take-th largest of the 256,
// `bound` (found by bisection on the key's bits, but for the lowest, each wavefront by itself).  All keys that reach it are
// gathered, about -256 ln(1 - take/256) whatever the row looks like where the columns are dealt out (127 for 100 winners,
// 355 for 192).  With block maxima the row itself is not read but for the about as many blocks that reach the bound, whose
// columns are dealt out for a second one (many of their keys can reach the first: a near list of which every vector is
// better than the best of the far ones).  The order of the keys follows from counting, for each, the ones before it.
// The k best of 78,000 scores (10M x 96, 32 probes, 16 queries) took two launches of 25 and 7 us that read every score.
// Bound by latency: a handful of dependent reads, so what counts is that each is one round for all threads.
// Otherwise (more winners, or more than kSelCand keys reach the bound) an exact radix search, four 8-bit digits,
// most significant first.
constexpr int kSelU = 8;        // groups of 64 columns loaded together by k_select
constexpr int kSelSmallU = 8;   // and by k_select_small beyond its registers
constexpr int kSelCand = 512;   // most keys the short cut of k_select orders
constexpr int kSelAll = 128;    // most columns of a row that is ordered whole (as for 512, the square of whose number that takes: probes of
                                // 2048 queries over 512 cells, 20 us with a bound for 128 columns and more, 33 without one)
constexpr int kSelHeld = 16;    // columns (or block maxima) a thread keeps in registers between its two passes
constexpr int kSelBlocks = 512; // most blocks it gathers from
constexpr int kSelOffs = 256;   // most probes whose offsets are staged in LDS

// Both kinds of selection below run over a row's values twice: for the largest of a thread's share, and for those that reach the bound.  A key
// made of every value, a range test and an address for each were about 26 vector instructions a value.  So values are compared as floats,
// two to an instruction the first time, keys are made of those that pass, and full rounds of loads do without range tests (10,000 queries
// at 10M x 96: k best of the nearest lists 68 -> 56 us, 32 of 4096 cells 61.5 -> 59.5, the call 600 -> 583; one query at 1M x 128 25.9 -> 25.5).
// Values that are no number have the lowest key and no part in the comparison of floats, but that a share of nothing else counts as -inf: such
// a bound may be reached by fewer keys than winners are wanted, and then the radix search takes over.
// A lower bound of the take-th largest of the 256 keys at `maxima`, less than 2^10 below it (0 when there are fewer).  For
// few winners of the 64 keys that are the largest of four each, which is another such bound and hardly lower (30 keys
// of a row dealt out reach it for 24 winners instead of 25) at a quarter of the steps.
__device__ __forceinline__ uint32_t kth_of_maxima(const uint32_t* maxima, int take, int lane) {
    const uint4 m4 = *reinterpret_cast<const uint4*>(maxima + 4 * lane);
    uint32_t bound = 0;
    if (take <= 24) {
        const uint32_t one = max(max(m4.x, m4.y), max(m4.z, m4.w));
        for (int bit = 31; bit >= 10; --bit) {
            const uint32_t test = bound | (1u << bit);
            if (__popcll(__ballot(one >= test)) >= take) bound = test;
        }
        return bound;
    }
    for (int bit = 31; bit >= 10; --bit) {
        const uint32_t test = bound | (1u << bit);
        const int cnt = __popcll(__ballot(m4.x >= test)) + __popcll(__ballot(m4.y >= test)) +
                        __popcll(__ballot(m4.z >= test)) + __popcll(__ballot(m4.w >= test));
        if (cnt >= take) bound = test;
    }
    return bound;
}

// COPIES: counters per digit in the histogram (a power of two; 8 pays for long rows, 1 for short ones, where
// clearing and summing the copies costs more than the collisions they avoid).
// SHORT: with the short cut, whose LDS and registers calls of more winners do without.
template <int MODE, int COPIES, bool SHORT>
__global__ __launch_bounds__(256) void k_select(SelectArgs a) {
    constexpr int kHistCopies = COPIES;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int32_t s_off[kSelOffs + 1];
    int kpad = 1;
    while (kpad < a.k) kpad <<= 1;
    // kHistCopies counters per digit, chosen by lane: keys of one row often share their leading byte, and
    // 64 lanes adding to one LDS word are served one after the other
    uint32_t* hist = reinterpret_cast<uint32_t*>(smem);               // [256][kHistCopies]
    uint32_t* ctrl = hist + 256 * kHistCopies;                        // [8]
    uint32_t* wave_cnt = ctrl + 8;                                    // [4]
    uint32_t* s_key = wave_cnt + 4;                                   // [kpad]
    uint32_t* s_col = s_key + kpad;                                   // [kpad]
    int64_t* s_lab = reinterpret_cast<int64_t*>(s_col + kpad);   // [kpad], 8-byte aligned: 268 + 2*kpad words
    uint64_t* c_ent = reinterpret_cast<uint64_t*>(s_lab + kpad);      // [kSelCand + 8] key << 32 | ~column of the short cut; before that its maxima ...
    int2* c_blk = reinterpret_cast<int2*>(c_ent + kSelCand + 8);      // [kSelBlocks] ... and the blocks that reach the bound

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t row = blockIdx.x;
    const float* vals = a.vals + row * a.stride;
    const int64_t q = row;
    const int32_t* off = MODE == 0 ? nullptr : a.cand_off + q * (a.np + 1);
    const int n_off = MODE == 0 ? 0 : a.p_limit ? a.p_limit[q] : a.np;
    const int m = MODE == 0 ? a.m_fixed : off[n_off];
    const bool staged = a.np <= kSelOffs;
    if (MODE == 1 && staged)
        for (int p = tid; p <= a.np; p += 256) s_off[p] = off[p];
    auto off_at = [&](int p) -> int32_t { return staged ? s_off[p] : off[p]; };
    const int k = a.k;
    const int take = m < k ? m : k;

    for (int i = tid; i < kpad; i += 256) { s_key[i] = 0u; s_col[i] = 0xFFFFFFFFu; s_lab[i] = INT64_MAX; }

    // each wavefront owns a contiguous quarter [w_begin, w_end) of the row
    const int chunk = ((m + 3) / 4 + 63) & ~63;
    const int w_begin = wave * chunk < m ? wave * chunk : m;
    const int w_end = (w_begin + chunk < m) ? w_begin + chunk : m;
    uint32_t prefix = 0, mask = 0;
    uint32_t need = (uint32_t)take;
    bool picked = false;
    if (tid == 0) { ctrl[5] = 0; ctrl[6] = 0; }
    const int n_blk = MODE == 1 && a.blk_max ? block_index(m, n_off) : 0;
    // (few blocks for many winners: their maxima say little.  100 winners of 12,000 candidates, 200 blocks: 34 us a call through the
    // blocks, 30 from the scores)
    const bool by_block = n_blk >= 2 * take && m > kSelCand;
    if (SHORT && take > 0 && ((take <= kSelTake && m > k) || m <= kSelAll)) {
        // (one base pointer and loads without a branch between them, so that all of a thread's are in flight together)
        const uint32_t* src = by_block ? a.blk_max + row * a.blk_stride : reinterpret_cast<const uint32_t*>(vals);
        const int parts = by_block ? n_blk : m;
        uint32_t* maxima = reinterpret_cast<uint32_t*>(c_ent);
        uint32_t held[kSelHeld], bound = 0;
        if (parts <= 1024) {
#pragma unroll
            for (int u = 0; u < 4; ++u) held[u] = src[min(256 * u + tid, parts - 1)];
        } else {
#pragma unroll
            for (int u = 0; u < kSelHeld; ++u) held[u] = src[min(256 * u + tid, parts - 1)];
        }
        auto read_on = [&](int i0, uint32_t (&v)[kSelU]) {
            if (i0 + 256 * kSelU <= parts) {
#pragma unroll
                for (int u = 0; u < kSelU; ++u) v[u] = (src + i0 + 256 * u)[(uint32_t)tid];
            } else {
#pragma unroll
                for (int u = 0; u < kSelU; ++u) v[u] = src[min(i0 + 256 * u + tid, parts - 1)];
            }
        };
        if (parts > kSelAll || by_block) {
            if (by_block) {
                uint32_t best = 0;
#pragma unroll
                for (int u = 0; u < kSelHeld; ++u) best = 256 * u + tid < parts ? max(best, held[u]) : best;
                for (int i0 = 256 * kSelHeld; i0 < parts; i0 += 256 * kSelU) {
                    uint32_t v[kSelU];
                    read_on(i0, v);
#pragma unroll
                    for (int u = 0; u < kSelU; ++u) best = i0 + 256 * u + tid < parts ? max(best, v[u]) : best;
                }
                maxima[tid] = best;
            } else {
                float best = -__builtin_inff();
                auto fold = [&](int i0, const uint32_t* v) {
                    if (i0 + 256 * kSelU <= parts) {
#pragma unroll
                        for (int u = 0; u < kSelU; u += 2) best = max3(best, __uint_as_float(v[u]), __uint_as_float(v[u + 1]));
                    } else {
#pragma unroll
                        for (int u = 0; u < kSelU; ++u)
                            best = i0 + 256 * u + tid < parts && __uint_as_float(v[u]) > best ? __uint_as_float(v[u]) : best;
                    }
                };
                static_assert(kSelHeld == 2 * kSelU, "two rounds held");
                fold(0, held);
                if (256 * kSelU < parts) fold(256 * kSelU, held + kSelU);
                for (int i0 = 256 * kSelHeld; i0 < parts; i0 += 256 * kSelU) {
                    uint32_t v[kSelU];
                    read_on(i0, v);
                    fold(i0, v);
                }
                maxima[tid] = tid < parts ? order_key(best) : 0u;
            }
            __syncthreads();
            bound = kth_of_maxima(maxima, take, lane);
        }
        __syncthreads();               // the maxima are no longer read: the entries take their place
        auto gather = [&](uint32_t key, int col) {
            const uint32_t pos = atomicAdd(&ctrl[5], 1u);
            if (pos < (uint32_t)kSelCand) c_ent[pos] = (uint64_t)key << 32 | (uint32_t)~col;
        };
        const float least = order_value(bound);          // (no number where there is no bound: every value goes on)
        auto pass = [&](uint32_t raw, int i) {
            if (!by_block) {
                if (__uint_as_float(raw) < least) return;
                const uint32_t key = order_key(__uint_as_float(raw));
                if (i < parts && key >= bound) gather(key, i);
            } else if (i < parts && raw >= bound) {
                const uint32_t pos = atomicAdd(&ctrl[6], 1u);
                if (pos < (uint32_t)kSelBlocks) c_blk[pos].x = i;
            }
        };
#pragma unroll
        for (int u = 0; u < kSelHeld; ++u) {
            if (256 * u >= parts) break;
            pass(held[u], 256 * u + tid);
        }
        for (int i0 = 256 * kSelHeld; i0 < parts; i0 += 256 * kSelU) {
            uint32_t v[kSelU];
            read_on(i0, v);
#pragma unroll
            for (int u = 0; u < kSelU; ++u) pass(v[u], i0 + 256 * u + tid);
        }
        __syncthreads();
        if (by_block && ctrl[6] <= (uint32_t)kSelBlocks) {
            const int n = (int)ctrl[6];
            // first column of a block, and how many it has
            for (int b = tid; b < n; b += 256) {
                const int i = c_blk[b].x;
                int lo = 0, hi = n_off;                 // largest p with block_index(off(p), p) <= i
                while (hi - lo > 1) {
                    const int mid = (lo + hi) >> 1;
                    if (block_index(off_at(mid), mid) <= i) lo = mid; else hi = mid;
                }
                const int c0 = off_at(lo) + (i - block_index(off_at(lo), lo)) * 64;
                c_blk[b] = make_int2(c0, off_at(lo + 1) - c0);
            }
            __syncthreads();
            // kSelHeld blocks of a wavefront at a time, the first of them kept in registers
            float v[kSelHeld];
            int col[kSelHeld];                          // (-1: none)
            auto read = [&](int b0) {
#pragma unroll
                for (int e = 0; e < kSelHeld; ++e) {
                    const int b = b0 + 4 * e;
                    const int2 c = c_blk[b < n ? b : 0];
                    col[e] = b < n && lane < c.y ? c.x + lane : -1;
                    v[e] = vals[max(col[e], 0)];
                }
            };
            auto for_keys = [&](auto use) {
                for (int b0 = wave; b0 < n; b0 += 4 * kSelHeld) {
                    if (b0 != wave || n > 4 * kSelHeld) read(b0);
#pragma unroll
                    for (int e = 0; e < kSelHeld; ++e) {
                        if (b0 + 4 * e >= n) break;
                        if (col[e] >= 0) use(order_key(v[e]), col[e]);
                    }
                }
            };
            read(wave);
            uint32_t best = 0;
            for_keys([&](uint32_t key, int) { best = max(best, key); });
            maxima[tid] = best;
            __syncthreads();
            bound = max(bound, kth_of_maxima(maxima, take, lane));
            __syncthreads();
            for_keys([&](uint32_t key, int c) { if (key >= bound) gather(key, c); });
            __syncthreads();
        }
        const int found = (int)ctrl[5];
        picked = found >= take && found <= kSelCand && (!by_block || ctrl[6] <= (uint32_t)kSelBlocks);      // uniform over the workgroup
        if (picked) {
            // place of every gathered key in (key desc, column asc) order
            // (the loads of eight entries in flight together: the loop is their latency and nothing else)
            if (tid < 8) c_ent[found + tid] = 0;
            __syncthreads();
            for (int i = tid; i < found; i += 256) {
                const uint64_t me = c_ent[i];
                int rank = 0;
                for (int j = 0; j < found; j += 8) {
                    uint64_t o[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) o[e] = c_ent[j + e];
#pragma unroll
                    for (int e = 0; e < 8; ++e) rank += o[e] > me ? 1 : 0;
                }
                if (rank < take) { s_key[rank] = (uint32_t)(me >> 32); s_col[rank] = ~(uint32_t)me; }
            }
        }
        __syncthreads();
    }
    if (picked) {
        // winners are in place
    } else if (take > 0 && m > k) {
        for (int pass = 0; pass < 4; ++pass) {
            const int shift = 24 - 8 * pass;
#pragma unroll
            for (int e = 0; e < kHistCopies; ++e) hist[tid + 256 * e] = 0;
            __syncthreads();
            // kSelU groups of 64 columns per step, their loads in flight together (the pass is bound by the
            // latency of reading the row, not by its arithmetic)
            for (int i0 = w_begin; i0 < w_end; i0 += 64 * kSelU) {
                float v[kSelU];
#pragma unroll
                for (int u = 0; u < kSelU; ++u) {
                    const int i = i0 + 64 * u + lane;
                    v[u] = vals[i < w_end ? i : w_end - 1];
                }
#pragma unroll
                for (int u = 0; u < kSelU; ++u) {
                    const uint32_t key = order_key(v[u]);
                    if (i0 + 64 * u + lane < w_end && (key & mask) == prefix)
                        atomicAdd(&hist[((key >> shift) & 255u) * kHistCopies + (lane & (kHistCopies - 1))], 1u);
                }
            }
            __syncthreads();
            if (wave == 0) {
                // the digit where the count of keys with larger digits first reaches `need`: lane l owns the
                // digits 4l .. 4l+3, a suffix sum over the lanes gives what lies above each lane
                uint32_t h[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    h[e] = 0;
#pragma unroll
                    for (int c = 0; c < kHistCopies; ++c) h[e] += hist[(lane * 4 + e) * kHistCopies + c];
                }
                const uint32_t own = h[0] + h[1] + h[2] + h[3];
                uint32_t incl = own;
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const uint32_t t = __shfl_down(incl, o);
                    if (lane + o < 64) incl += t;
                }
                uint32_t above = incl - own;
                int found = -1;
                uint32_t before = 0;
#pragma unroll
                for (int e = 3; e >= 0; --e) {
                    if (found < 0 && above < need && above + h[e] >= need) { found = lane * 4 + e; before = above; }
                    above += h[e];
                }
                if (found >= 0) { ctrl[0] = (uint32_t)found; ctrl[1] = need - before; }   // exactly one lane (need >= 1)
            }
            __syncthreads();
            prefix |= ctrl[0] << shift;
            mask |= 255u << shift;
            need = ctrl[1];
            __syncthreads();
        }
    } else {
        need = 0;   // everything is taken (m <= k): threshold below every key
    }
    // now: keys > prefix are all kept (take - need of them); `need` of the keys == prefix are kept
    const bool all = !(take > 0 && m > k);
    if (tid == 0) { ctrl[2] = 0; ctrl[3] = 0; }
    __syncthreads();
    const uint32_t n_above = (uint32_t)take - need;
    if (take > 0 && !picked) {
        // Keys above the threshold go anywhere in the first n_above places (atomic counter).  Keys equal to it
        // are taken in column order: each wavefront owns a contiguous quarter of the row, counts its ties in a
        // first sweep and, once the counts of the wavefronts before it are known, places them in a second.
        uint32_t my_ties = 0;
        for (int i0 = w_begin; i0 < w_end; i0 += 64 * kSelU) {
            float v[kSelU];
#pragma unroll
            for (int u = 0; u < kSelU; ++u) {
                const int i = i0 + 64 * u + lane;
                v[u] = vals[i < w_end ? i : w_end - 1];
            }
#pragma unroll
            for (int u = 0; u < kSelU; ++u) {
                const int i = i0 + 64 * u + lane;
                const uint32_t key = order_key(v[u]);
                const bool above = i < w_end && (all || key > prefix);
                const bool tie = i < w_end && !all && key == prefix;
                if (above) {
                    const uint32_t pos = atomicAdd(&ctrl[2], 1u);
                    s_key[pos] = key;
                    s_col[pos] = (uint32_t)i;
                }
                my_ties += (uint32_t)__popcll(__ballot(tie));
            }
        }
        if (lane == 0) wave_cnt[wave] = my_ties;
        __syncthreads();
        uint32_t before = 0;
        for (int w = 0; w < wave; ++w) before += wave_cnt[w];
        for (int i0 = w_begin; i0 < w_end && before < need && my_ties > 0; i0 += 64) {
            const int i = i0 + lane;
            uint32_t key = 0;
            bool tie = false;
            if (i < w_end) {
                key = order_key(vals[i]);
                tie = !all && key == prefix;
            }
            const uint64_t bal = __ballot(tie);
            const uint32_t rank = before + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
            if (tie && rank < need) {
                s_key[n_above + rank] = key;
                s_col[n_above + rank] = (uint32_t)i;
            }
            before += (uint32_t)__popcll(bal);
        }
    }
    __syncthreads();

    // labels
    for (int i = tid; i < take; i += 256) {
        const uint32_t col = s_col[i];
        if (MODE == 0) {
            s_lab[i] = (int64_t)col;
        } else {
            int lo = 0, hi = n_off;         // largest p with off[p] <= col
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (off_at(mid) <= (int32_t)col) lo = mid; else hi = mid;
            }
            const int l = a.probe[q * a.np + lo];
            const int64_t slot = a.list_off[l] + ((int32_t)col - off_at(lo));
            s_lab[i] = a.ids ? a.ids[slot] : slot;       // without a label table the slot itself is the result
        }
    }
    __syncthreads();

    // order by (key desc, label asc); empty entries (key 0, label max) sink
    auto put = [&](int i, uint32_t key, int64_t lab) {
        const bool real = i < take && key != 0u;
        float v = real ? order_value(key) : -__builtin_inff();
        if (MODE == 1 && a.metric) v = metric_value(a.metric, v, a.qnorm[q]);
        if (a.out_vals) a.out_vals[row * k + i] = v;
        if (MODE == 0) { if (a.out_i32) a.out_i32[row * k + i] = real ? (int32_t)lab : -1; }
        else { if (a.out_i64) a.out_i64[row * k + i] = real ? lab : -1; }
        if (MODE == 0) s_col[i] = real ? (uint32_t)lab : 0xFFFFFFFFu;
    };
    if (kpad <= 256 && picked) {
        const uint32_t key = tid < take ? s_key[tid] : 0u;
        // (the short cut's winners are in this order already but for equal keys; counting orders those.  Winners of the radix search
        // are in no order: 200 of them counted made a call of 10,000 queries x 2500 candidates 445 us, 409 with the network below)
        const bool tie = tid + 1 < take && key == s_key[tid + 1];
        if (__syncthreads_or(tie)) {
            const int64_t lab = tid < kpad ? s_lab[tid] : 0;
            int rank = tid;                          // an empty place
            if (tid < take) {
                rank = 0;
#pragma unroll 4
                for (int j = 0; j < take; ++j) {
                    const uint32_t kj = s_key[j];
                    const int64_t lj = s_lab[j];
                    rank += (int)(kj > key) | ((int)(kj == key) & ((int)(lj < lab) | ((int)(lj == lab) & (int)(j < tid))));
                }
            }
            if (tid < k) put(rank, key, lab);
        } else if (tid < k) {
            put(tid, key, s_lab[tid]);
        }
    } else {
        for (int size = 2; size <= kpad; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                for (int i = tid; i < kpad / 2; i += 256) {
                    const int lo_i = 2 * i - (i & (stride - 1));
                    const int hi_i = lo_i + stride;
                    const bool up = ((lo_i & size) == 0);
                    const uint32_t k0 = s_key[lo_i], k1 = s_key[hi_i];
                    const int64_t l0 = s_lab[lo_i], l1 = s_lab[hi_i];
                    const bool first_before = (k0 > k1) || (k0 == k1 && l0 <= l1);   // lo already precedes hi
                    if (first_before != up) {
                        s_key[lo_i] = k1; s_key[hi_i] = k0;
                        s_lab[lo_i] = l1; s_lab[hi_i] = l0;
                    }
                }
                __syncthreads();
            }
        }
        for (int i = tid; i < k; i += 256) put(i, s_key[i], s_lab[i]);
    }
    // mode 0: the candidate offsets follow from the probes, which are in LDS (the running sums take the place of the labels)
    if (MODE == 0 && a.cand.cand_off) {
        __syncthreads();
        if (wave == 0) cand_offsets_wave(a.cand, row, k, reinterpret_cast<const int32_t*>(s_col), reinterpret_cast<int32_t*>(s_lab), lane);
    }
}

// ---- selection for short rows: one wavefront per row ------------------------------------------
//
// For rows of at most kSmallM values (bound known to the host) and k <= 64 a wavefront does the whole selection on its own,
// without workgroup barriers: the k-th largest key is found by a four-pass radix search (8 bits per
// pass, a 256-bin histogram private to the wavefront, a suffix sum over the lanes), then the values
// above it and, in column order, as many equal to it as are still needed are compacted with
// ballots.  The first 64*NV columns of the row are loaded once, all loads in flight together, and
// every pass takes them from registers; columns beyond that (long rows are rare) are re-read from
// memory in each pass.  A wavefront needs little LDS, so many rows are in flight per compute unit.  A final bitonic pass over the lanes orders the winners by (value desc, label asc).

constexpr int kSmallM = 16384;
constexpr int kShortcutTake = 32;     // the lane-maxima short cut pays up to this many winners (beyond, too many keys reach the bound)

// WIDE: the instantiation for more than kShortcutTake winners (its second short cut costs the common case of
// fewer winners a fifth of its speed when both sit in one kernel).
template <int MODE, int NV, bool WIDE = false>
// (probe selection, MODE 0, is held to the registers of four wavefronts per SIMD: 10,000 rows over 4096 cells
// take 0.072 ms so, 0.100 ms at the two wavefronts its unconstrained register count allows; the result rows of
// MODE 1 lose from the same limit)
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(MODE == 0 ? 4 : 1, 8))) void k_select_small(SelectArgs a) {
    __shared__ uint32_t s_work[4][256 + 64];             // per wavefront: 256 bins, 64 winning columns
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t row = (int64_t)blockIdx.x * 4 + wave;
    if (row >= a.rows) return;
    const int64_t q = row;
    const int m = MODE == 0 ? a.m_fixed : a.cand_off[q * (a.np + 1) + (a.p_limit ? a.p_limit[q] : a.np)];
    const int k = a.k;
    const int take = m < k ? m : k;
    const float* vals = a.vals + row * a.stride;
    uint32_t* hist = s_work[wave];                                      // [256]
    int* win_col = reinterpret_cast<int*>(hist + 256);                  // [64]
    const float ninf = -__builtin_inff();
    auto key_of = [](float v) -> uint32_t { return order_key(v); };

    win_col[lane] = -1;
    float held[NV];                                      // column e*64 + lane (unused beyond m)
    if (NV * 64 <= m) {
#pragma unroll
        for (int e = 0; e < NV; ++e) held[e] = (vals + e * 64)[(uint32_t)lane];
    } else {
#pragma unroll
        for (int e = 0; e < NV; ++e) held[e] = vals[e * 64 + lane < m ? e * 64 + lane : 0];
    }
    auto read_on = [&](int i0, float (&v)[kSelSmallU]) {
        if (i0 + 64 * kSelSmallU <= m) {
#pragma unroll
            for (int u = 0; u < kSelSmallU; ++u) v[u] = (vals + i0 + 64 * u)[(uint32_t)lane];
        } else {
#pragma unroll
            for (int u = 0; u < kSelSmallU; ++u) { const int i = i0 + 64 * u + lane; v[u] = vals[i < m ? i : m - 1]; }
        }
    };
    // the largest of N columns' values and of `best`, every STEP-th of them from column FIRST on
    auto fold = [&](auto n, auto first, auto step, int i0, const float* v, float best) {
        constexpr int N = decltype(n)::value, FIRST = decltype(first)::value, STEP = decltype(step)::value;
        if (i0 + 64 * N <= m) {
#pragma unroll
            for (int e = FIRST; e < N; e += 2 * STEP) best = max3(best, v[e], v[e + STEP]);
        } else {
#pragma unroll
            for (int e = FIRST; e < N; e += STEP) best = i0 + 64 * e + lane < m && v[e] > best ? v[e] : best;
        }
        return best;
    };
    const std::integral_constant<int, NV> all{};
    const std::integral_constant<int, kSelSmallU> more{};
    const std::integral_constant<int, 0> c0{};
    const std::integral_constant<int, 1> c1{};
    const std::integral_constant<int, 2> c2{};

    // Short cut.  The take-th largest of the 64 lane maxima is reached by at least `take` keys (one per lane
    // that holds such a maximum), so every winner is among the keys that reach it; there are seldom many more
    // than `take` of them.  When at most 64 do, they are compacted into the lanes, sorted by (key desc, column
    // asc) and the first `take` are the winners: the same set as the radix search below would pick.
    bool done = false;
    if (take > 0 && take <= kShortcutTake) {
        float lane_max = fold(all, c0, c1, 0, held, ninf);
        for (int i0 = NV * 64; i0 < m; i0 += 64 * kSelSmallU) {
            float v[kSelSmallU];
            read_on(i0, v);
            lane_max = fold(more, c0, c1, i0, v, lane_max);
        }
        uint32_t sorted = lane < m ? key_of(lane_max) : 0u;                      // the lane maxima in descending order over the lanes
#pragma unroll
        for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                const uint32_t other = __shfl_xor(sorted, stride);
                const bool lower = (lane & stride) == 0, up = (lane & size) == 0;
                const bool keep = (lower == up) ? (sorted >= other) : (sorted <= other);
                sorted = keep ? sorted : other;
            }
        }
        const uint32_t reach = __shfl(sorted, take - 1);
        if (reach != 0u) {
            uint32_t* c_key = hist;                      // [64] keys that reach it, [64] their columns
            int* c_col = reinterpret_cast<int*>(hist + 64);
            uint32_t count = 0;
            const float least = order_value(reach);
            auto collect = [&](int i, float v) {
                if (__ballot(!(v < least)) == 0) return;
                const uint32_t key = key_of(v);
                const bool in = i < m && key >= reach;
                const uint64_t b = __ballot(in);
                const uint32_t pos = count + (uint32_t)__popcll(b & (((uint64_t)1 << lane) - 1));
                if (in && pos < 64u) { c_key[pos] = key; c_col[pos] = i; }
                count += (uint32_t)__popcll(b);
            };
#pragma unroll
            for (int e = 0; e < NV; ++e)
                if (e * 64 < m) collect(e * 64 + lane, held[e]);
            for (int i0 = NV * 64; i0 < m && count <= 64u; i0 += 64 * kSelSmallU) {
                float v[kSelSmallU];
                read_on(i0, v);
#pragma unroll
                for (int u = 0; u < kSelSmallU; ++u)
                    if (i0 + 64 * u < m) collect(i0 + 64 * u + lane, v[u]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (count >= (uint32_t)take && count <= 64u) {
                uint32_t ck = lane < (int)count ? c_key[lane] : 0u;
                int cc = lane < (int)count ? c_col[lane] : INT32_MAX;
#pragma unroll
                for (int size = 2; size <= 64; size <<= 1) {
#pragma unroll
                    for (int stride = size >> 1; stride > 0; stride >>= 1) {
                        const uint32_t ok = __shfl_xor(ck, stride);
                        const int oc = __shfl_xor(cc, stride);
                        const bool lower = (lane & stride) == 0, up = (lane & size) == 0;
                        const bool mine_first = (ck > ok) || (ck == ok && cc <= oc);
                        const bool keep = (lower == up) ? mine_first : !mine_first;
                        if (!keep) { ck = ok; cc = oc; }
                    }
                }
                if (lane < take) win_col[lane] = cc;
                done = true;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();         // the words of `hist` are free again
        }
    }
    // The same idea for up to 64 winners, with two maxima per lane (over the even and over the odd 64-column
    // blocks of the row): the take-th largest of these 128 is again reached by at least `take` keys, and by few
    // more.  It is found by bisection on the key's bits (two ballots a bit); up to 128 keys that reach it are
    // compacted into LDS and every one counts the keys that precede it in (key desc, column asc) order, which is
    // its place among the winners.
    if (WIDE && !done && take > kShortcutTake && take <= 64) {
        static_assert(NV % 4 == 0 && kSelSmallU % 4 == 0, "pairs of blocks of either parity");
        float max0 = fold(all, c0, c2, 0, held, ninf), max1 = fold(all, c1, c2, 0, held, ninf);
        for (int i0 = NV * 64; i0 < m; i0 += 64 * kSelSmallU) {
            float v[kSelSmallU];
            read_on(i0, v);
            max0 = fold(more, c0, c2, i0, v, max0);
            max1 = fold(more, c1, c2, i0, v, max1);
        }
        const uint32_t gm0 = lane < m ? key_of(max0) : 0u, gm1 = lane + 64 < m ? key_of(max1) : 0u;
        uint32_t reach = 0u;
        for (int bit = 31; bit >= 0; --bit) {
            const uint32_t test = reach | (1u << bit);
            const int cnt = __popcll(__ballot(gm0 >= test)) + __popcll(__ballot(gm1 >= test));
            if (cnt >= take) reach = test;
        }
        if (reach != 0u) {
            uint32_t* c_key = hist;                      // [128] keys that reach it, [128] their columns
            int* c_col = reinterpret_cast<int*>(hist + 128);
            uint32_t count = 0;
            const float least = order_value(reach);
            auto collect = [&](int i, float v) {
                if (__ballot(!(v < least)) == 0) return;
                const uint32_t key = key_of(v);
                const bool in = i < m && key >= reach;
                const uint64_t b = __ballot(in);
                const uint32_t pos = count + (uint32_t)__popcll(b & (((uint64_t)1 << lane) - 1));
                if (in && pos < 128u) { c_key[pos] = key; c_col[pos] = i; }
                count += (uint32_t)__popcll(b);
            };
#pragma unroll
            for (int e = 0; e < NV; ++e)
                if (e * 64 < m) collect(e * 64 + lane, held[e]);
            for (int i0 = NV * 64; i0 < m && count <= 128u; i0 += 64 * kSelSmallU) {
                float v[kSelSmallU];
                read_on(i0, v);
#pragma unroll
                for (int u = 0; u < kSelSmallU; ++u)
                    if (i0 + 64 * u < m) collect(i0 + 64 * u + lane, v[u]);
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            if (count >= (uint32_t)take && count <= 128u) {
                const int n_c = (int)count;
                const bool has0 = lane < n_c, has1 = lane + 64 < n_c;
                const uint32_t k0 = has0 ? c_key[lane] : 0u, k1 = has1 ? c_key[lane + 64] : 0u;
                const int c0 = has0 ? c_col[lane] : 0, c1 = has1 ? c_col[lane + 64] : 0;
                int r0 = 0, r1 = 0;
                for (int jj = 0; jj < n_c; ++jj) {
                    const uint32_t kj = c_key[jj];
                    const int cj = c_col[jj];
                    r0 += (kj > k0 || (kj == k0 && cj < c0)) ? 1 : 0;
                    r1 += (kj > k1 || (kj == k1 && cj < c1)) ? 1 : 0;
                }
                if (has0 && r0 < take) win_col[r0] = c0;
                if (has1 && r1 < take) win_col[r1] = c1;
                done = true;
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();         // the words of `hist` are free again
        }
    }
    if (!done) {
    uint32_t keys[NV];
#pragma unroll
    for (int e = 0; e < NV; ++e) keys[e] = key_of(held[e]);
    // radix search for the take-th largest key
    uint32_t prefix = 0, mask = 0, need = (uint32_t)take;
    // Leading bytes that every key of the row shares (scores of one query usually share sign and exponent)
    // need no pass: their histogram would be one bin that all lanes hit at once.
    int top_shift = 24;
    if (take > 0) {
        const uint32_t first = __builtin_amdgcn_readfirstlane(keys[0]);
        uint32_t diff = 0u;
#pragma unroll
        for (int e = 0; e < NV; ++e) diff |= (e * 64 + lane < m) ? (keys[e] ^ first) : 0u;
        for (int i0 = NV * 64; i0 < m; i0 += 64 * kSelSmallU) {                               // columns beyond the registers,
            float v[kSelSmallU];                                                               // kSelSmallU loads in flight together
#pragma unroll
            for (int u = 0; u < kSelSmallU; ++u) { const int i = i0 + 64 * u + lane; v[u] = vals[i < m ? i : m - 1]; }
#pragma unroll
            for (int u = 0; u < kSelSmallU; ++u) diff |= key_of(v[u]) ^ first;                  // a clamped column repeats the last one
        }
        if (__ballot((diff >> 24) != 0u) == 0ull) {
            prefix = first & 0xFF000000u; mask = 0xFF000000u; top_shift = 16;
            if (__ballot((diff >> 16) != 0u) == 0ull) { prefix = first & 0xFFFF0000u; mask = 0xFFFF0000u; top_shift = 8; }
        }
    }
    if (take > 0) {
        for (int shift = top_shift; shift >= 0; shift -= 8) {
#pragma unroll
            for (int e = 0; e < 4; ++e) hist[lane * 4 + e] = 0u;
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int e = 0; e < NV; ++e)
                if (e * 64 + lane < m && (keys[e] & mask) == prefix) atomicAdd(&hist[(keys[e] >> shift) & 255u], 1u);
            for (int i0 = NV * 64; i0 < m; i0 += 64 * kSelSmallU) {
                float v[kSelSmallU];
#pragma unroll
                for (int u = 0; u < kSelSmallU; ++u) { const int i = i0 + 64 * u + lane; v[u] = vals[i < m ? i : m - 1]; }
#pragma unroll
                for (int u = 0; u < kSelSmallU; ++u) {
                    const uint32_t key = key_of(v[u]);
                    if (i0 + 64 * u + lane < m && (key & mask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            // lane l owns digits 4l .. 4l+3; above = how many keys have a digit beyond this lane's
            uint32_t h[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) h[e] = hist[lane * 4 + e];
            const uint32_t own = h[0] + h[1] + h[2] + h[3];
            uint32_t incl = own;                                     // inclusive suffix sum over lanes
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const uint32_t t = __shfl_down(incl, o);
                if (lane + o < 64) incl += t;
            }
            uint32_t above = incl - own;
            // the digit where the running count first reaches `need`, scanning digits downwards
            int found = -1;
            uint32_t before = 0;
#pragma unroll
            for (int e = 3; e >= 0; --e) {
                if (found < 0 && above < need && above + h[e] >= need) { found = lane * 4 + e; before = above; }
                above += h[e];
            }
            const uint64_t who = __ballot(found >= 0);               // exactly one lane while need >= 1
            const int src = who ? (int)__builtin_ctzll(who) : 0;
            const int dgt = __shfl(found, src);
            before = __shfl(before, src);
            need -= before;
            prefix |= (uint32_t)dgt << shift;
            mask |= 255u << shift;
        }
    }
    // keys above the threshold, then `need` keys equal to it in column order
    const uint32_t n_above = (uint32_t)take - need;
    uint32_t base_gt = 0, base_eq = 0;
    auto place = [&](int i, uint32_t key) {
        const bool gt = i < m && key > prefix;
        const bool eq = i < m && key == prefix;
        const uint64_t bg = __ballot(gt), be = __ballot(eq);
        const uint64_t below = ((uint64_t)1 << lane) - 1;
        if (gt) win_col[base_gt + (uint32_t)__popcll(bg & below)] = i;
        const uint32_t rank_eq = base_eq + (uint32_t)__popcll(be & below);
        if (eq && rank_eq < need) win_col[n_above + rank_eq] = i;
        base_gt += (uint32_t)__popcll(bg);
        base_eq += (uint32_t)__popcll(be);
    };
    if (take > 0) {
#pragma unroll
        for (int e = 0; e < NV; ++e)
            if (e * 64 < m) place(e * 64 + lane, keys[e]);
        for (int i0 = NV * 64; i0 < m; i0 += 64 * kSelSmallU) {
            float v[kSelSmallU];
#pragma unroll
            for (int u = 0; u < kSelSmallU; ++u) { const int i = i0 + 64 * u + lane; v[u] = vals[i < m ? i : m - 1]; }
#pragma unroll
            for (int u = 0; u < kSelSmallU; ++u)
                if (i0 + 64 * u < m) place(i0 + 64 * u + lane, key_of(v[u]));
        }
    }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int out_c = lane < take ? win_col[lane] : -1;
    float out_v = out_c >= 0 ? vals[out_c] : ninf;

    // labels, then order equal values by label
    int64_t lab = INT64_MAX;
    if (out_c >= 0) {
        lab = MODE == 0 ? out_c : 0;      // (mode 1: a placeholder, resolved below by the whole wavefront)
    }
    if (MODE == 1) {
        // probe rank of each winner: the last p with cand_off[p] <= column.  Up to 256 probes the row of
        // offsets is staged in the wavefront's LDS words (the histogram is no longer needed) and every
        // winner bisects there; beyond that the offsets are handed round with shuffles, 64 at a time.
        const int32_t* off = a.cand_off + q * (a.np + 1);
        int rank = 0, rank_off = 0;
        if (a.np <= 256) {
            int32_t* s_off = reinterpret_cast<int32_t*>(hist);
            for (int p = lane; p < a.np; p += 64) s_off[p] = off[p];
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            int lo = 0, hi = a.np;               // off[0] = 0 <= column
            while (hi - lo > 1) {
                const int mid = (lo + hi) >> 1;
                if (s_off[mid] <= out_c) lo = mid; else hi = mid;
            }
            rank = lo;
            rank_off = s_off[lo];
        } else {
            for (int base = 0; base < a.np; base += 64) {
                const int p = base + lane;
                const int32_t mine_off = p < a.np ? off[p] : INT32_MAX;
                const int span = a.np - base < 64 ? a.np - base : 64;
                for (int t = 0; t < span; ++t) {
                    const int32_t o = __shfl(mine_off, t);
                    if (o <= out_c) { rank = base + t; rank_off = o; }
                }
            }
        }
        if (out_c >= 0) {
            const int64_t slot = a.list_off[a.probe[q * a.np + rank]] + (out_c - rank_off);
            lab = a.ids ? a.ids[slot] : slot;
        }
    }
    // order the winners by (value desc, label asc): a bitonic network over the first nsort >= take lanes
    // (the others hold nothing); the value travels as its key and is decoded at the end
    uint32_t key = out_c >= 0 ? key_of(out_v) : 0u;
    const int nsort = take <= 8 ? 8 : take <= 16 ? 16 : take <= 32 ? 32 : 64;
#pragma unroll
    for (int size = 2; size <= 64; size <<= 1) {
        if (size > nsort) break;
#pragma unroll
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const uint32_t ok = __shfl_xor(key, stride);
            const int64_t ol = __shfl_xor(lab, stride);
            const bool lower = (lane & stride) == 0;     // this lane holds the earlier position of the pair
            const bool up = (lane & size) == 0;          // block sorted into final order (best first)
            const bool mine_first = (key > ok) || (key == ok && lab <= ol);
            const bool keep = (lower == up) ? mine_first : !mine_first;
            if (!keep) { key = ok; lab = ol; }
        }
    }
    out_v = order_value(key);
    if (lane < k) {
        const bool real = key != 0u;
        if (a.out_vals) a.out_vals[row * k + lane] = real ? out_v : ninf;
        if (MODE == 0) { if (a.out_i32) a.out_i32[row * k + lane] = real ? (int32_t)lab : -1; }
        else { if (a.out_i64) a.out_i64[row * k + lane] = real ? lab : -1; }
    }
    // MODE 0: the candidate offsets follow from the probes while the lanes still hold them (with a launch of their own,
    // which reads the probes back, a search of one query over 1M x 128 takes 45.2 us, so 43.9)
    if (MODE == 0 && a.cand.cand_off) cand_offsets_lanes(a.cand, row, k, key != 0u ? (int)lab : -1, lane);
}

// ---- re-ranking on raw vectors (Section "Architecture", Search: optional) -----------------------
//
// One workgroup per query: each wavefront takes every fourth candidate and computes <q, x> / (|q| |x|) from the raw
// rows, then the workgroup orders by (score desc, label asc) and emits the k best, dropping repeated labels.  Bound by
// the latency of gathering rows: a wavefront reads the labels of its next 64 candidates together and then four rows together
// (T: coordinates of a lane); 4096 queries x 50 rows of 128: 63 us with one row at a time and a sort by one barrier a step, 40 now.
// Up to 256 candidates are placed by counting the ones that go before (by the wavefronts that have one: by all four, the
// reads of LDS alone made it 100 us), more are sorted.  4096 queries x 100 coordinates, sorted by one barrier a step, one row at
// a time, against now: 50 candidates 63 and 40 us, 128 113 and 84, 200 210 and 158, 256 225 and 180, 300 (sorted) 391 and 257; one
// query, 256 candidates 55 and 34 (62 with && and || in the counting loops).  The labels have to lie at multiples of 8: 4 bytes off, 200
// candidates took 284 us, 256 315.
template <int T>
__global__ __launch_bounds__(256) void k_rerank(RerankArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int U = 4;
    int size = 1;
    while (size < a.r) size <<= 1;
    int64_t* s_lab = reinterpret_cast<int64_t*>(smem);
    uint32_t* s_key = reinterpret_cast<uint32_t*>(s_lab + size);
    float* s_val = reinterpret_cast<float*>(s_key + size);
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float* qv = a.q + q * a.d;
    float qr[T];
    float qq = 0.f;
#pragma unroll
    for (int e = 0; e < T; ++e) {
        const int j = lane + 64 * e;
        qr[e] = j < a.d ? qv[j] : 0.f;
        qq += qr[e] * qr[e];
    }
    qq = wave_sum(qq);
    for (int c64 = wave; c64 < size; c64 += 4 * 64) {
        const int c_own = c64 + 4 * lane;
        const int64_t own = c_own < a.r ? a.cand[q * a.r + c_own] : -1;
        const int many = (size - c64 + 3) / 4 < 64 ? (size - c64 + 3) / 4 : 64;
        for (int m = 0; m < many; m += U) {
            float v[U][T];
            int64_t id[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)own, m + u);
                const int hi = __builtin_amdgcn_readlane((int)(own >> 32), m + u);
                id[u] = (int64_t)hi << 32 | lo;
                if (id[u] >= a.n_rows) id[u] = -1;
                const float* xv = id[u] >= 0 ? a.x + id[u] * a.d : qv;       // (no such row: the query's own is read and not used)
#pragma unroll
                for (int e = 0; e < T; ++e) {
                    const int j = lane + 64 * e;
                    v[u][e] = xv[j < a.d ? j : a.d - 1];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int c = c64 + 4 * (m + u);
                float xy = 0.f, xx = 0.f;
#pragma unroll
                for (int e = 0; e < T; ++e) {
                    if (lane + 64 * e >= a.d) v[u][e] = 0.f;
                    xy += v[u][e] * qr[e];
                    xx += v[u][e] * v[u][e];
                }
                xy = wave_sum(xy);
                xx = wave_sum(xx);
                if (lane == 0 && c < size) {
                    const bool ok = id[u] >= 0 && xx > 0.f && qq > 0.f;
                    const float sc = ok ? xy / sqrtf(xx * qq) : -__builtin_inff();
                    s_key[c] = ok ? order_key(sc) : 0u;
                    s_val[c] = sc;
                    s_lab[c] = ok ? id[u] : INT64_MAX;
                }
            }
        }
    }
    if (size <= 256) {
        __shared__ int s_out;
        if (tid == 0) s_out = 0;
        __syncthreads();
        const uint32_t key = tid < a.r ? s_key[tid] : 0u;
        const int64_t lab = tid < a.r ? s_lab[tid] : INT64_MAX;
        // the same label again has the same score: all but the first are taken out
        const int look = 64 * wave < a.r ? a.r : 0;        // (a wavefront without a candidate places none)
        int again = 0;       // (no && and || around the reads of LDS: each is a branch and a wait of its own)
#pragma unroll 8
        for (int i = 0; i < look; ++i) again |= (int)(i < tid) & (int)(s_lab[i] == lab);
        __syncthreads();
        const bool counts = key != 0u && !again;
        if (tid < a.r && !counts) s_key[tid] = 0u;
        if (counts) atomicAdd(&s_out, 1);
        __syncthreads();
        int place = 0;
#pragma unroll 8
        for (int i = 0; i < look; ++i) {
            const uint32_t ki = s_key[i];
            place += (int)(ki > key) | ((int)(ki == key) & (int)(s_lab[i] < lab));
        }
        if (counts && place < a.k) {
            a.out_scores[q * a.k + place] = s_val[tid];
            a.out_ids[q * a.k + place] = lab;
        }
        for (int i = s_out + tid; i < a.k; i += 256) { a.out_scores[q * a.k + i] = -__builtin_inff(); a.out_ids[q * a.k + i] = -1; }
        return;
    }
    __syncthreads();
    for (int sz = 2; sz <= size; sz <<= 1) {
        for (int stride = sz >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < size / 2; i += 256) {
                const int lo_i = 2 * i - (i & (stride - 1));
                const int hi_i = lo_i + stride;
                const bool up = ((lo_i & sz) == 0);
                const uint32_t k0 = s_key[lo_i], k1 = s_key[hi_i];
                const int64_t l0 = s_lab[lo_i], l1 = s_lab[hi_i];
                const bool first_before = (k0 > k1) || (k0 == k1 && l0 <= l1);
                if (first_before != up) {
                    s_key[lo_i] = k1; s_key[hi_i] = k0;
                    s_lab[lo_i] = l1; s_lab[hi_i] = l0;
                    const float v0 = s_val[lo_i]; s_val[lo_i] = s_val[hi_i]; s_val[hi_i] = v0;
                }
            }
            __syncthreads();
        }
    }
    if (tid == 0) {
        int out = 0;
        int64_t prev = INT64_MAX;
        for (int i = 0; i < size && out < a.k; ++i) {
            if (s_key[i] == 0u) break;
            if (s_lab[i] == prev) continue;                  // the same label again: equal score, adjacent
            prev = s_lab[i];
            a.out_scores[q * a.k + out] = s_val[i];
            a.out_ids[q * a.k + out] = s_lab[i];
            ++out;
        }
        for (; out < a.k; ++out) { a.out_scores[q * a.k + out] = -__builtin_inff(); a.out_ids[q * a.k + out] = -1; }
    }
}

// ---- cascade search, pass 2 (Appendix "Cascade search via Lloyd-Max bin ordinality") ------------
//
// One workgroup per query.  Each wavefront takes kept candidates in turn: finds the probed list that
// holds the slot (lanes over the query's probes), then lane j sums the coordinates j, j+64, ... from
// the packed words; the workgroup sorts (score desc, label asc) in LDS and emits the k best.
__global__ __launch_bounds__(256) void k_cascade_rescore(CascadeArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    int size = 1;
    while (size < a.n_keep) size <<= 1;
    uint32_t* s_key = reinterpret_cast<uint32_t*>(smem);
    float* s_val = reinterpret_cast<float*>(s_key + size);
    int64_t* s_lab = reinterpret_cast<int64_t*>(s_val + size);
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t mask = (1u << a.b) - 1u;
    float zr[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int j = lane + 64 * e;
        zr[e] = j < a.d ? a.z[q * a.z_pitch + j] : 0.f;
    }
    for (int c = wave; c < size; c += 4) {
        const int64_t slot = c < a.n_keep ? a.cand[q * a.n_keep + c] : -1;
        int p_found = -1;
        if (slot >= 0) {
            for (int base = 0; base < a.np && p_found < 0; base += 64) {
                const int p = base + lane;
                bool hit = false;
                if (p < a.np) {
                    const int l = a.probe[q * a.np + p];
                    const int64_t off = l < 0 ? 0 : a.store.list_off[l];
                    hit = l >= 0 && slot >= off && slot < off + a.store.list_size[l];
                }
                const unsigned long long m = __ballot(hit);
                if (m) p_found = base + __ffsll((long long)m) - 1;
            }
        }
        float acc = 0.f;
        if (p_found >= 0) {
            const uint32_t* wp = a.store.codes + (slot >> 6) * a.store.words * 64 + (slot & 63);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int j = lane + 64 * e;
                if (j < a.d) {
                    const int bit = j * a.b, w = bit >> 5, o = bit & 31;
                    uint32_t v = wp[(int64_t)w * 64] >> o;
                    if (o + a.b > 32) v |= wp[(int64_t)(w + 1) * 64] << (32 - o);
                    acc += zr[e] * a.cb[v & mask];
                }
            }
        }
        for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o);
        if (lane == 0) {
            const bool ok = p_found >= 0;
            float sc = -__builtin_inff();
            if (ok) sc = a.coarse[q * a.np + p_found] + __half2float(__ushort_as_half(a.store.gamma[slot])) * acc;
            s_key[c] = ok ? order_key(sc) : 0u;
            s_val[c] = sc;
            s_lab[c] = ok ? a.ids[slot] : INT64_MAX;
        }
    }
    __syncthreads();
    for (int sz = 2; sz <= size; sz <<= 1) {
        for (int stride = sz >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < size / 2; i += 256) {
                const int lo_i = 2 * i - (i & (stride - 1));
                const int hi_i = lo_i + stride;
                const bool up = ((lo_i & sz) == 0);
                const uint32_t k0 = s_key[lo_i], k1 = s_key[hi_i];
                const int64_t l0 = s_lab[lo_i], l1 = s_lab[hi_i];
                const bool first_before = (k0 > k1) || (k0 == k1 && l0 <= l1);
                if (first_before != up) {
                    s_key[lo_i] = k1; s_key[hi_i] = k0;
                    s_lab[lo_i] = l1; s_lab[hi_i] = l0;
                    const float v0 = s_val[lo_i]; s_val[lo_i] = s_val[hi_i]; s_val[hi_i] = v0;
                }
            }
            __syncthreads();
        }
    }
    for (int i = tid; i < a.k; i += 256) {
        const bool real = i < size && s_key[i] != 0u;
        a.out_scores[q * a.k + i] = real ? s_val[i] : -__builtin_inff();
        a.out_ids[q * a.k + i] = real ? s_lab[i] : -1;
    }
}

}  // namespace

hipError_t launch_cascade_rescore(const CascadeArgs& a, int64_t nq, hipStream_t st) {
    if (nq <= 0) return hipSuccess;
    int size = 1;
    while (size < a.n_keep) size <<= 1;
    const size_t lds = (size_t)size * 16;
    hipLaunchKernelGGL(k_cascade_rescore, dim3((unsigned)nq), dim3(256), lds, st, a);
    return hipGetLastError();
}

hipError_t launch_rerank(const RerankArgs& a, int64_t nq, hipStream_t st) {
    if (nq <= 0) return hipSuccess;
    int size = 1;
    while (size < a.r) size <<= 1;
    const size_t lds = (size_t)size * 16;
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)nq), dim3(256), lds, st, a); };
    switch ((a.d + 63) / 64) {
        case 1: go(k_rerank<1>); break;
        case 2: go(k_rerank<2>); break;
        case 3: go(k_rerank<3>); break;
        default: go(k_rerank<4>); break;
    }
    return hipGetLastError();
}

hipError_t launch_list_scan(const ListScanArgs& a, int b, int64_t q_count, int blocks_per_query, int slices, hipStream_t st) {
    if (q_count <= 0) return hipSuccess;
    if (a.metric && (!a.qnorm || !a.store.xnorm)) return hipErrorInvalidValue;
    const size_t lut_bytes = (size_t)a.d * (1u << b) * sizeof(float);
    const bool direct = lut_bytes > 64 * 1024;
    size_t lds = direct ? (size_t)(a.d + (1 << b)) * sizeof(float) : lut_bytes;
    if (a.gate) lds = std::max(lds, kRedoLds);
    // slices: every list is dealt out in rounds of 256 vectors to that many workgroups (grid z, the slowest
    // dimension of the dispatch order: the launch works through the index one slice at a time)
    dim3 grid((unsigned)(blocks_per_query > 0 ? blocks_per_query : a.np), (unsigned)q_count, (unsigned)std::max(1, std::min(slices, 64)));
    if (a.gate) grid = dim3(kRedoWorkgroups);
    if (a.gate && (a.k < 1 || a.k > kRedoSort || a.gate_rows < std::min(a.gate_count, kRedoWorkgroups))) return hipErrorInvalidValue;
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(a.gate ? kRedoThreads : 256), lds, st, a); };
#define IVFTQ_SCAN(BV)                                                                              \
    case BV:                                                                                        \
        if (a.gate) direct ? go(k_list_scan<BV, true, true, false>) : go(k_list_scan<BV, false, true, false>);                \
        else if (a.blk_max) direct ? go(k_list_scan<BV, true, false, true>) : go(k_list_scan<BV, false, false, true>);        \
        else direct ? go(k_list_scan<BV, true, false, false>) : go(k_list_scan<BV, false, false, false>);                      \
        break;
    switch (b) {
        IVFTQ_SCAN(1) IVFTQ_SCAN(2) IVFTQ_SCAN(3) IVFTQ_SCAN(4)
        IVFTQ_SCAN(5) IVFTQ_SCAN(6) IVFTQ_SCAN(7) IVFTQ_SCAN(8)
        default: return hipErrorInvalidValue;
    }
#undef IVFTQ_SCAN
    return hipGetLastError();
}

// Longest row the one-wavefront-per-row kernel takes, for up to 64 winners: of cells (mode 0, every row has m_fixed) and of
// results (mode 1, mostly much shorter than their bound).
constexpr int kSmallMax0 = 8192, kSmallMax1 = kSmallM;
// Up to that many rows of at most m values a workgroup each is faster all the same, the launch being bound by the latency of one row.
// Coarse scores and probe selection together, 32 coordinates, 32 probes, workgroup and wavefront, us: 1024 queries x 512 cells 16.0 and
// 15.7, 1000 cells 15.8 and 16.1, 4096 cells 24.3 and 29.6; 2048 queries x 512 cells 20.0 and 17.3, 1000 cells 22.6 and 19.2, 2000 cells 28.0
// and 25.9, 4096 cells 35.8 and 37.7; 10,000 queries x 1000 cells 61.5 and 39.1 (x 4096 90.4 and 95.8: the line could lie higher there).
constexpr int64_t few_rows(int m) { return m <= 2048 ? 1024 : 2048; }
hipError_t launch_select(int mode, const SelectArgs& a, hipStream_t st) {
    if (a.rows <= 0) return hipSuccess;
    // short rows and small k: the one-wavefront-per-row kernel
    const int m_bound = mode == 0 ? a.m_fixed : a.m_bound;
    const bool small = a.k <= 64 && m_bound > 0 && m_bound <= (mode == 0 ? kSmallMax0 : kSmallMax1);
    if (small && !a.blk_max && a.rows > few_rows(m_bound)) {
        const dim3 blocks((unsigned)((a.rows + 3) / 4));
        const bool wide = a.k > kShortcutTake;
        const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, blocks, dim3(256), 0, st, a); };
        if (mode == 1) wide ? go(k_select_small<1, 16, true>) : go(k_select_small<1, 16>);
        else if (m_bound <= 1536) wide ? go(k_select_small<0, 16, true>) : go(k_select_small<0, 16>);
        else wide ? go(k_select_small<0, 32, true>) : go(k_select_small<0, 32>);
        return hipGetLastError();
    }
    int kpad = 1;
    while (kpad < a.k) kpad <<= 1;
    const int copies = (m_bound == 0 || m_bound > 8192) ? 8 : 1;
    // Long rows of which more are wanted than the short cut takes: its LDS and registers cost a workgroup of five on a compute unit.  Selection
    // with them and without, us: 753 of 345,657 for 1150 queries 2294 and 1757, 1000 of 28,000 222 and 150.  (Rows of up to 8192 keep the
    // form for all: those of at most 128 are ordered whole.)
    const bool plain = copies == 8 && a.k > kSelTake;
    const size_t lds = (256 * copies + 8 + 4) * 4 + (size_t)kpad * 16 + (plain ? 0 : (size_t)(kSelCand + 8 + kSelBlocks) * 8);
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3((unsigned)a.rows), dim3(256), lds, st, a); };
    if (plain) mode == 0 ? go(k_select<0, 8, false>) : go(k_select<1, 8, false>);
    else if (copies == 8) mode == 0 ? go(k_select<0, 8, true>) : go(k_select<1, 8, true>);
    else mode == 0 ? go(k_select<0, 1, true>) : go(k_select<1, 1, true>);
    return hipGetLastError();
}

}  // namespace ivftq
