// Query-batched list scan on the matrix cores (Section "Architecture", Search: the residual
// estimate gamma * <Pi q~, C[code]> for every vector of every probed list): everything around the scan
// kernel itself (batch_scan.h).
//
// In a large query batch each inverted list is probed by many queries (Q * nprobe / nlist of them
// on average), so the scan of one list against all of its queries is a dense contraction:
// [vectors of the list] x [d] times [d] x [queries probing the list].  The (query, probe) pairs are
// regrouped by list here, a wavefront of the scan takes a part of one list and a tile of its queries, scores that reach the
// query's threshold (the k-th best score of its nearest lists, found beforehand) land in a short per-query
// candidate list, and the merge puts those and the nearest lists' k best together.
#include <hip/hip_fp16.h>

#include "kernels.h"

namespace ivftq {

namespace {

// ---- regrouping (query, probe) pairs by list ---------------------------------------------------
//
// Pairs are bucketed with atomic counters: bucket l holds the pairs (q, p < first[q]) of list l
// (each query's nearest lists, scanned first to find its threshold), bucket L + l the others.  The order of the pairs inside a bucket (and so
// which tile a query lands in) may change from run to run; results do not, because a score depends
// only on its own (query, vector) pair and the final merge orders candidates by (score, label).

__global__ void k_pair_count(const int32_t* __restrict__ probe, const int32_t* __restrict__ first, int64_t nq,
                             int np, int L, uint32_t* __restrict__ count) {
    const int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (it >= nq * np) return;
    const int late = (int)(it % np) >= first[it / np];
    if (probe[it] >= 0) atomicAdd(&count[probe[it] + (late ? L : 0)], 1u);      // (no cell: a query whose scores are no numbers)
}

// Every bucket gets a range of the pair array (pair_off) and of its pass's tile array, its record, and
// cursor[b] = 0.  One thread per bucket; a workgroup puts its buckets together with a scan and takes its ranges from
// the totals with one atomic each, so the ranges of different workgroups lie in no particular order, which nothing
// depends on (in bucket order, by one workgroup: 0.017 ms for 8192 buckets, the chain of its loads).  A thread writes the first kOwnTiles
// tiles of its bucket, wavefronts the rest: a few long lists that meet many queries have a thousand and more each (33 lists, 9699
// queries x 5 probes: 44 us by a thread each, 14 so).
constexpr uint32_t kOwnTiles = 64;
__global__ __launch_bounds__(256) void k_pair_ranges(const int32_t* __restrict__ list_size, const int64_t* __restrict__ list_off, int nb,
                                                     int L, TileShape shape, PairTable p) {
    __shared__ uint32_t part[4][3];
    __shared__ int32_t start[3];
    __shared__ int4 many[256];
    __shared__ int n_many;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, b = (int)blockIdx.x * 256 + tid;
    if (tid == 0) n_many = 0;
    const bool in = b < nb, near = b < L;
    const uint32_t n = in ? p.count[b] : 0u;
    const int size = in ? list_size[near ? b : b - L] : 0;
    const int64_t slot = in ? list_off[near ? b : b - L] : 0;
    if (in) p.cursor[b] = 0u;
    const uint32_t w = near ? shape.tq_near : shape.tq;
    const uint32_t tiles = size > 0 ? (n + w - 1) / w * list_parts(size, near ? shape.part_near : shape.part) : 0u;
    const uint32_t own[3] = {n, near ? tiles : 0u, near ? 0u : tiles};
    uint32_t incl[3] = {own[0], own[1], own[2]};
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const uint32_t v = __shfl_up(incl[i], o);
            if (lane >= o) incl[i] += v;
        }
    if (lane == 63)
#pragma unroll
        for (int i = 0; i < 3; ++i) part[wave][i] = incl[i];
    __syncthreads();
    if (tid < 3) start[tid] = atomicAdd(&p.totals[tid], (int32_t)(part[0][tid] + part[1][tid] + part[2][tid] + part[3][tid]));
    __syncthreads();
    int32_t at[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        at[i] = start[i] + (int32_t)(incl[i] - own[i]);
        for (int w2 = 0; w2 < wave; ++w2) at[i] += (int32_t)part[w2][i];
    }
    const int32_t t0 = near ? at[1] : at[2];
    int32_t* to = near ? p.tile_near : p.tile_late;
    if (in) {
        p.pair_off[b] = at[0];
        int4* rec = reinterpret_cast<int4*>(p.record + (int64_t)b * kPairRecord);
        rec[0] = make_int4(size, t0, (int)n, at[0]);
        rec[1] = make_int4((int)(uint32_t)slot, (int)(slot >> 32), 0, 0);
        for (uint32_t t = 0; t < min(tiles, kOwnTiles); ++t) to[t0 + t] = b;
    }
    // the others of the buckets with more: a wavefront a bucket
    if (tiles > kOwnTiles) many[atomicAdd(&n_many, 1)] = make_int4(t0, (int)tiles, b, 0);
    __syncthreads();
    for (int i = wave; i < n_many; i += 4) {
        const int4 m = many[i];
        int32_t* at_bucket = (m.z < L ? p.tile_near : p.tile_late) + m.x;
        for (int t = (int)kOwnTiles + lane; t < m.y; t += 64) at_bucket[t] = m.z;
    }
}

__global__ void k_pair_scatter(const int32_t* __restrict__ probe, const int32_t* __restrict__ first, int64_t nq,
                               int np, int L, const int32_t* __restrict__ pair_off,
                               uint32_t* __restrict__ cursor, int32_t* __restrict__ pairs) {
    const int64_t it = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (it >= nq * np) return;
    const int late = (int)(it % np) >= first[it / np];
    const int bkt = probe[it] + (late ? L : 0);
    if (probe[it] >= 0) pairs[pair_off[bkt] + atomicAdd(&cursor[bkt], 1u)] = (int32_t)it;
}

// The second step alone, where the probe selection has counted the pairs and left each one's place in its bucket.  (Counting in a launch of
// its own and a second round of updates of the buckets took 9 us more for 1000 queries x 16 probes, 20 for 10,000 x 64.)
__global__ __launch_bounds__(256) void k_pair_place(const int32_t* __restrict__ probe, const int32_t* __restrict__ first, const int32_t* __restrict__ rank,
                                                    int64_t n, int np, int L, const int32_t* __restrict__ pair_off, int32_t* __restrict__ pairs) {
    const int64_t it = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (it >= n) return;
    const int l = probe[it], at = rank[it], q = (int)it / np;
    if (l >= 0) pairs[pair_off[l + ((int)it - q * np >= first[q] ? L : 0)] + at] = (int32_t)it;
}

// Both steps with the counters privatised in LDS: a workgroup takes kPairChunk consecutive
// pairs, counts them per bucket in LDS, and touches each global counter once per bucket it met
// (thousands of pairs hit the same few thousand counters, so per-pair global atomics serialise).
// In the scatter step that one global atomic reserves the workgroup's range inside the bucket.
constexpr int kPairChunk = 4096;
constexpr int kPairLdsBuckets = 16384;      // 2L must not exceed this (64 KB of LDS)

__global__ __launch_bounds__(1024) void k_pair_count_lds(const int32_t* __restrict__ probe,
                                                         const int32_t* __restrict__ first, int64_t nq, int np,
                                                         int L, uint32_t* __restrict__ count) {
    extern __shared__ uint32_t bins[];                   // [2L]
    for (int i = threadIdx.x; i < 2 * L; i += 1024) bins[i] = 0u;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * kPairChunk, total = nq * np;
    const int64_t end = begin + kPairChunk < total ? begin + kPairChunk : total;
    for (int64_t it = begin + threadIdx.x; it < end; it += 1024) {
        const int late = (int)(it % np) >= first[it / np];
        if (probe[it] >= 0) atomicAdd(&bins[probe[it] + (late ? L : 0)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * L; i += 1024)
        if (bins[i]) atomicAdd(&count[i], bins[i]);
}

__global__ __launch_bounds__(1024) void k_pair_scatter_lds(const int32_t* __restrict__ probe,
                                                           const int32_t* __restrict__ first, int64_t nq, int np,
                                                           int L, const int32_t* __restrict__ pair_off,
                                                           uint32_t* __restrict__ cursor, int32_t* __restrict__ pairs) {
    extern __shared__ uint32_t bins[];                   // [2L] count, then first position of this workgroup's range
    for (int i = threadIdx.x; i < 2 * L; i += 1024) bins[i] = 0u;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * kPairChunk, total = nq * np;
    const int64_t end = begin + kPairChunk < total ? begin + kPairChunk : total;
    for (int64_t it = begin + threadIdx.x; it < end; it += 1024) {
        const int late = (int)(it % np) >= first[it / np];
        if (probe[it] >= 0) atomicAdd(&bins[probe[it] + (late ? L : 0)], 1u);
    }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * L; i += 1024) {
        const uint32_t c = bins[i];
        bins[i] = c ? atomicAdd(&cursor[i], c) : 0u;      // this workgroup's pairs of bucket i start here
    }
    __syncthreads();
    for (int64_t it = begin + threadIdx.x; it < end; it += 1024) {
        const int late = (int)(it % np) >= first[it / np];
        const int bkt = probe[it] + (late ? L : 0);
        if (probe[it] >= 0) pairs[pair_off[bkt] + atomicAdd(&bins[bkt], 1u)] = (int32_t)it;
    }
}


// ---- merge: first-pass top-k and threshold-pass candidates -> the k best --------------------------
//
// One workgroup per query.  First-pass entries carry exact scores; a candidate carries an upper bound u of its score,
// the score itself lying in [lo, u], lo = u - 2*kappa*gamma (times the factor by which a raw metric scales scores).
// At least k entries have lower bounds of R or more for the k-th largest lower bound R, so an entry with u < R is
// not among the k best.  R need not be exact: the lower bounds are counted in 256 equal bins between the k-th
// first-pass score (itself such a bound) and the largest, and an entry survives when its u falls into the bin that
// holds the k-th largest lower bound, or a higher one (binning never decreases, so u in a lower bin means u < R).
// The survivors, a few more than k, are re-scored from the packed codes in float32, 16 lanes each, and placed by
// counting, for every one, those that precede it in (score desc, label asc) order.  A query whose candidate list
// overflowed is appended to the gate list.  Bound by latency: passes over a few hundred values in LDS and one
// dependent gather per survivor.  (Sorting all entries by u, then the survivors by score: 0.21 ms instead of
// 0.13 for 4096 queries with 385 candidates each, k = 50.)
// (0: no number, which is no result)
__device__ __forceinline__ uint32_t okey(float f) {
    const uint32_t u = __float_as_uint(f);
    return f != f ? 0u : (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__device__ __forceinline__ float okey_value(uint32_t k) { return __uint_as_float((k & 0x80000000u) ? (k ^ 0x80000000u) : ~k); }

constexpr int kMergeCount = 256;        // most survivors placed by counting; beyond that a bitonic network sorts them

__global__ __launch_bounds__(256) void k_merge(MergeArgs a) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t hist[256];
    __shared__ float s_wmax[4];
    __shared__ int s_bin, s_found;
    const int64_t q = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int cnt = a.cand_cnt[q];
    if (cnt > a.cap) {                           // the exact pass redoes this query
        if (tid == 0) a.gate[1 + atomicAdd(&a.gate[0], 1)] = (int32_t)q;
        return;
    }
    const float qn = a.metric ? a.qnorm[q] : 1.f;
    auto put = [&](int i, float key, int64_t lab) {
        a.out_scores[q * a.k + i] = a.metric ? metric_value(a.metric, key, qn) : key;
        a.out_ids[q * a.k + i] = lab;
    };
    if (cnt == 0) {                              // nothing beat the threshold: the first pass's k best stand as they are
        for (int i = tid; i < a.k; i += 256) put(i, a.first_scores[q * a.k + i], a.first_ids[q * a.k + i]);
        return;
    }
    const int total = a.k + cnt;
    int size = 1;
    while (size < total) size <<= 1;
    int64_t* p_lab = reinterpret_cast<int64_t*>(smem);               // [size] survivors: label, before re-scoring the packed slot
    float* s_u = reinterpret_cast<float*>(p_lab + size);             // [total] upper bounds
    uint32_t* p_key = reinterpret_cast<uint32_t*>(s_u + total);      // [size] survivors: entry number, then key of the score
    float* s_z = reinterpret_cast<float*>(p_key + size);             // [d] the query's rotated coordinates
    float* s_cb = s_z + a.d;                                         // [2^b]
    for (int j = tid; j < a.d; j += 256) s_z[j] = a.z[q * a.z_pitch + j];
    for (int j = tid; j < (1 << a.b); j += 256) s_cb[j] = a.cb[j];
    hist[tid] = 0;
    if (tid == 0) { s_bin = 0; s_found = 0; }
    constexpr int64_t kSlotMask = ((int64_t)1 << kCandProbeShift) - 1;
    constexpr int kHeld = 8;                     // lower bounds of a thread's first entries, kept between the two passes
    float held[kHeld];
    float top = -__builtin_inff();
    auto bounds = [&](int i, float& lo) -> float {
        if (i < a.k) return lo = a.first_scores[q * a.k + i];
        const float u = a.cand_score[q * a.cap + (i - a.k)];
        const int64_t slot = a.cand_slot[q * a.cap + (i - a.k)] & kSlotMask;
        const float g = __half2float(__ushort_as_half(a.store.gamma[slot]));
        lo = u - 2.f * a.kappa * g * (a.metric ? metric_scale(a.metric, a.store.xnorm[slot], qn) : 1.f);
        return u;
    };
#pragma unroll
    for (int h = 0; h < kHeld; ++h) {
        const int i = tid + 256 * h;
        held[h] = -__builtin_inff();
        if (i < total) s_u[i] = bounds(i, held[h]);
        top = fmaxf(top, held[h]);
    }
    for (int i = tid + 256 * kHeld; i < total; i += 256) {
        float lo;
        s_u[i] = bounds(i, lo);
        top = fmaxf(top, lo);
    }
    for (int o = 32; o > 0; o >>= 1) top = fmaxf(top, __shfl_xor(top, o));
    if (lane == 0) s_wmax[wave] = top;
    __syncthreads();
    top = fmaxf(fmaxf(s_wmax[0], s_wmax[1]), fmaxf(s_wmax[2], s_wmax[3]));
    const float base = s_u[a.k - 1];             // the k-th first-pass score (-inf when there are fewer)
    const float span = top - base;
    const bool binned = base > -__builtin_inff() && span > 0.f && span < __builtin_inff();
    const float scale = binned ? 255.f / span : 0.f;
    auto bin_of = [&](float v) -> int {          // -1: below the base
        const float x = (v - base) * scale;
        return v < base ? -1 : x < 255.f ? (int)x : 255;
    };
    auto count_bin = [&](float lo) {             // (the lower bound of an infinite norm is no number and counts for nothing)
        if (lo >= base) atomicAdd(&hist[bin_of(lo)], 1u);
    };
    if (binned) {
#pragma unroll
        for (int h = 0; h < kHeld; ++h) {
            if (tid + 256 * h >= total) break;
            count_bin(held[h]);
        }
        for (int i = tid + 256 * kHeld; i < total; i += 256) {
            float lo;
            (void)bounds(i, lo);
            count_bin(lo);
        }
    }
    __syncthreads();
    if (binned && wave == 0) {                   // the highest bin that at least k lower bounds reach
        uint32_t h[4], own = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) { h[e] = hist[4 * lane + e]; own += h[e]; }
        uint32_t above = own;                    // suffix sum over the lanes
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t t = __shfl_down(above, o);
            if (lane + o < 64) above += t;
        }
        above -= own;
        int found = -1;
#pragma unroll
        for (int e = 3; e >= 0; --e) {
            above += h[e];
            if (found < 0 && above >= (uint32_t)a.k) found = 4 * lane + e;
        }
        if (found >= 0) atomicMax(&s_bin, found);
    }
    __syncthreads();
    const int low_bin = s_bin;
    for (int i = tid; i < total; i += 256) {
        const bool missing = i < a.k && a.first_ids[q * a.k + i] < 0;
        if (!missing && (!binned || bin_of(s_u[i]) >= low_bin)) p_key[atomicAdd(&s_found, 1)] = (uint32_t)i;
    }
    __syncthreads();
    // exact scores and labels of the survivors
    const int found = s_found;
    const uint32_t mask = (1u << a.b) - 1u;
    const int grp = tid >> 4, gl = tid & 15;
    for (int s = grp; s < found; s += 16) {
        const int i = (int)p_key[s];
        float sc;
        int64_t lab;
        if (i < a.k) {
            sc = s_u[i];
            lab = a.first_ids[q * a.k + i];
        } else {
            const int64_t packed = a.cand_slot[q * a.cap + (i - a.k)];
            const int64_t slot = packed & kSlotMask;
            const int pr = (int)(packed >> kCandProbeShift);
            const float g = __half2float(__ushort_as_half(a.store.gamma[slot]));
            const float base_sc = a.coarse[q * a.np + pr];
            const float xn = a.metric ? a.store.xnorm[slot] : 1.f;
            lab = a.ids ? a.ids[slot] : slot;
            const uint32_t* wp = a.store.codes + (slot >> 6) * a.store.words * 64 + (slot & 63);
            float acc = 0.f;
#pragma unroll 4
            for (int j = gl; j < a.d; j += 16) {
                const int bit = j * a.b, w = bit >> 5, o = bit & 31;
                uint32_t v = wp[(int64_t)w * 64] >> o;
                if (o + a.b > 32) v |= wp[(int64_t)(w + 1) * 64] << (32 - o);
                acc += s_z[j] * s_cb[v & mask];
            }
            for (int o = 8; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 16);
            sc = base_sc + g * acc;
            if (a.metric) sc = metric_key(a.metric, sc, xn, qn);
        }
        if (gl == 0) {
            p_key[s] = okey(sc);
            p_lab[s] = lab;
        }
    }
    __syncthreads();
    for (int i = found + tid; i < a.k; i += 256) put(i, -__builtin_inff(), -1);
    auto put_key = [&](int i, uint32_t key, int64_t lab) { put(i, key ? okey_value(key) : -__builtin_inff(), key ? lab : -1); };
    if (found <= kMergeCount) {
        if (tid < found) {
            const uint32_t key = p_key[tid];
            const int64_t lab = p_lab[tid];
            int rank = 0;
            for (int j = 0; j < found; ++j) {
                const uint32_t kj = p_key[j];
                const int64_t lj = p_lab[j];
                rank += (kj > key || (kj == key && (lj < lab || (lj == lab && j < tid)))) ? 1 : 0;
            }
            if (rank < a.k) put_key(rank, key, lab);
        }
        return;
    }
    int psize = 1;
    while (psize < found) psize <<= 1;
    for (int i = found + tid; i < psize; i += 256) { p_key[i] = 0u; p_lab[i] = INT64_MAX; }
    __syncthreads();
    for (int sz = 2; sz <= psize; sz <<= 1)
        for (int stride = sz >> 1; stride > 0; stride >>= 1) {
            for (int i = tid; i < psize / 2; i += 256) {
                const int lo_i = 2 * i - (i & (stride - 1)), hi_i = lo_i + stride;
                const uint32_t k0 = p_key[lo_i], k1 = p_key[hi_i];
                const int64_t l0 = p_lab[lo_i], l1 = p_lab[hi_i];
                if ((k0 > k1 || (k0 == k1 && l0 <= l1)) != ((lo_i & sz) == 0)) {
                    p_key[lo_i] = k1; p_key[hi_i] = k0;
                    p_lab[lo_i] = l1; p_lab[hi_i] = l0;
                }
            }
            __syncthreads();
        }
    for (int i = tid; i < a.k && i < found; i += 256) put_key(i, p_key[i], p_lab[i]);
}

}  // namespace

// The split float16 operands of the dense pass carry a level to 2^-23.  Over few terms, or with four levels that recur all
// the time, that rounding does not average out: root mean square error of the returned scores against float64, next to
// the streaming scan's, 1.03 at d = 10 and 1.02 at d = 32 with 2 bits, 1.02 at d = 8 with 4 and at d = 12 with 3, but 0.93
// to 0.99 at d = 16 to 32 with 3 or more bits and below that with more coordinates (0.82 at d = 256).
bool batch_covers(int d, int b) { return d >= 16 && d <= kMaxD && ((b >= 3 && b <= 5) || b == 8 || (b == 2 && d > 32)); }

hipError_t launch_pair_grouping(const int32_t* probe, const int32_t* first, const int32_t* rank, int64_t nq, int np, int L, const int32_t* list_size, const int64_t* list_off,
                                const TileShape& shape, const PairTable& p, hipStream_t st) {
    const int64_t n = nq * np;
    if (n <= 0) return hipSuccess;
    const auto ranges = [&] {
        hipLaunchKernelGGL(k_pair_ranges, dim3((unsigned)((2 * L + 255) / 256)), dim3(256), 0, st, list_size, list_off, 2 * L, L, shape, p);
    };
    if (rank) {
        ranges();
        hipLaunchKernelGGL(k_pair_place, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, probe, first, rank, n, np, L, (const int32_t*)p.pair_off, p.pairs);
        return hipGetLastError();
    }
    const bool in_lds = 2 * L <= kPairLdsBuckets;
    const unsigned blocks = (unsigned)(in_lds ? (n + kPairChunk - 1) / kPairChunk : (n + 255) / 256);
    const size_t lds = (size_t)2 * L * sizeof(uint32_t);
    if (in_lds) {
        static LdsLimit lim_count, lim_scatter;
        const size_t most = (size_t)kPairLdsBuckets * sizeof(uint32_t);
        hipError_t e = lim_count.ensure(reinterpret_cast<const void*>(k_pair_count_lds), most);
        if (e == hipSuccess) e = lim_scatter.ensure(reinterpret_cast<const void*>(k_pair_scatter_lds), most);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k_pair_count_lds, dim3(blocks), dim3(1024), lds, st, probe, first, nq, np, L, p.count);
        ranges();
        hipLaunchKernelGGL(k_pair_scatter_lds, dim3(blocks), dim3(1024), lds, st, probe, first, nq, np, L, (const int32_t*)p.pair_off, p.cursor, p.pairs);
    } else {
        hipLaunchKernelGGL(k_pair_count, dim3(blocks), dim3(256), 0, st, probe, first, nq, np, L, p.count);
        ranges();
        hipLaunchKernelGGL(k_pair_scatter, dim3(blocks), dim3(256), 0, st, probe, first, nq, np, L, (const int32_t*)p.pair_off, p.cursor, p.pairs);
    }
    return hipGetLastError();
}

hipError_t launch_batch_scan(const BatchScanArgs& a, int d, int b, hipStream_t st) {
    if (a.metric && (!a.qnorm || !a.store.xnorm)) return hipErrorInvalidValue;
    switch (b) {
        case 2: return batch_scan_b2(a, batch_dp(d), st);
        case 3: return batch_scan_b3(a, batch_dp(d), st);
        case 4: return batch_scan_b4(a, batch_dp(d), st);
        case 5: return batch_scan_b5(a, batch_dp(d), st);
        case 8: return batch_scan_b8(a, batch_dp(d), st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_merge(const MergeArgs& a, int64_t nq, hipStream_t st) {
    if (nq <= 0) return hipSuccess;
    int size = 1;
    while (size < a.k + a.cap) size <<= 1;
    const size_t lds = (size_t)size * 12 + (size_t)(a.k + a.cap + a.d + (1 << a.b)) * sizeof(float);
    static LdsLimit lim;
    const hipError_t e = lim.ensure(reinterpret_cast<const void*>(k_merge), 128 * 1024);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_merge, dim3((unsigned)nq), dim3(256), lds, st, a);
    return hipGetLastError();
}

}  // namespace ivftq
