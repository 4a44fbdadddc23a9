// Inverted-list bookkeeping for appends (Section "Architecture": "new vectors enter at any
// time"; Section "Streaming Experiments": append-only ingest with constant coarse parameters) and
// the centroid-update half of coarse k-means (Section "Architecture", Indexing).
//
// An append must place row i of the batch at position (old size of its list) + (number of earlier
// batch rows of the same list), so that list order equals arrival order and results never depend
// on scheduling.  That is a stable counting sort by cell number, done in three small kernels:
// per-segment histograms, a column-wise running sum over segments, and an in-order rank inside
// each segment by one workgroup.
#include <hip/hip_fp16.h>

#include <algorithm>

#include "kernels.h"
#include "split_f16.h"
#include "wave_sum.h"

namespace ivftq {

namespace {

__global__ __launch_bounds__(1024) void k_segment_hist(const int32_t* __restrict__ assign, int64_t n,
                                                       int64_t seg_len, int L, uint32_t* __restrict__ seg_hist) {
    extern __shared__ uint32_t hist[];
    for (int l = threadIdx.x; l < L; l += 1024) hist[l] = 0;
    __syncthreads();
    const int64_t begin = (int64_t)blockIdx.x * seg_len;
    const int64_t end = begin + seg_len < n ? begin + seg_len : n;
    for (int64_t i = begin + threadIdx.x; i < end; i += 4096) {          // four loads in flight
        int a[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) a[u] = i + 1024 * u < end ? assign[i + 1024 * u] : -1;
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (a[u] >= 0 && a[u] < L) atomicAdd(&hist[a[u]], 1u);
    }
    __syncthreads();
    for (int l = threadIdx.x; l < L; l += 1024) seg_hist[(int64_t)blockIdx.x * L + l] = hist[l];
}

// Column-wise exclusive running sum over segments.  A workgroup takes 16 lists; its 1024 threads split the
// segments into 64 parts (a sixteen-lane group per part) of at most kMaxSegments / 64, which a thread keeps in
// registers, all its loads in flight; a launch has L/16 workgroups.  batch_count may be host memory that the device can
// write, and flag a word that goes behind the counts there: the host waits for the kernel and nothing else.  (With two copies here, which are
// launches of their own, and one more for the new sizes after the encoding, 20,000 rows built and searched took 131 to 135 us, 97 to 103 now, on another machine 110 and 102.)
__global__ __launch_bounds__(1024) void k_segment_scan(uint32_t* __restrict__ seg_hist, int nseg, int L,
                                                       uint32_t* __restrict__ batch_count, const int* __restrict__ flag, int* __restrict__ flag_out) {
    if (flag && blockIdx.x == 0 && threadIdx.x == 0) *flag_out = *flag;
    constexpr int C = kMaxSegments / 64;
    __shared__ uint32_t part_sum[64][16];
    const int li = threadIdx.x & 15, part = threadIdx.x >> 4;
    const int l = blockIdx.x * 16 + li;
    const int chunk = (nseg + 63) / 64;
    const int s0 = part * chunk < nseg ? part * chunk : nseg;
    const int s1 = (s0 + chunk < nseg) ? s0 + chunk : nseg;
    uint32_t v[C], sum = 0;
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] = l < L && s0 + c < s1 ? seg_hist[(int64_t)(s0 + c) * L + l] : 0u;
#pragma unroll
    for (int c = 0; c < C; ++c) sum += v[c];
    part_sum[part][li] = sum;
    __syncthreads();
    uint32_t run = 0;
    for (int p = 0; p < part; ++p) run += part_sum[p][li];
    if (l < L) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            if (s0 + c < s1) seg_hist[(int64_t)(s0 + c) * L + l] = run;
            run += v[c];
        }
        if (part == 63) batch_count[l] = run;
    }
}

// A workgroup walks its segment 1024 rows at a time.  Its sixteen wavefronts find the equal cell numbers among
// their own 64 rows on their own, then add to the segment's counters in turn, in row order.  Bound by latency: a turn
// is one LDS atomic (the first row of a cell in a wavefront adds for all of them) and a barrier; the next rows'
// cell numbers are fetched before the turns.  (One wavefront per segment, segments of 128 rows: as many counters as
// 64 MB at 500,000 rows x 4096 cells, written once, read twice: the sort took 111 us an iteration of k-means.)
__global__ __launch_bounds__(kRankRows) void k_stable_rank(const int32_t* __restrict__ assign, int64_t n,
                                                           int64_t seg_len, int L,
                                                           const uint32_t* __restrict__ seg_hist,
                                                           const int64_t* __restrict__ list_base,
                                                           int64_t* __restrict__ slot,
                                                           const int64_t* __restrict__ batch_base,
                                                           int32_t* __restrict__ order, int2* __restrict__ order_cell,
                                                           const int32_t* __restrict__ new_size, int32_t* __restrict__ list_size) {
    extern __shared__ uint32_t cnt[];
    if (new_size && blockIdx.x == 0)
        for (int l = threadIdx.x; l < L; l += kRankRows) list_size[l] = new_size[l];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t begin = (int64_t)blockIdx.x * seg_len;
    const int64_t end = begin + seg_len < n ? begin + seg_len : n;
    int next = begin + threadIdx.x < end ? assign[begin + threadIdx.x] : -1;
    for (int l = threadIdx.x; l < L; l += kRankRows) cnt[l] = seg_hist[(int64_t)blockIdx.x * L + l];
    __syncthreads();
    const int nbits = 32 - __builtin_clz((unsigned)L);                      // bits of the numbers 0 .. L
    for (int64_t g = begin; g < end; g += kRankRows) {
        const int64_t i = g + threadIdx.x;
        const int key = next >= L ? -1 : next;
        next = i + kRankRows < end ? assign[i + kRankRows] : -1;
        // lanes holding the same cell number: one ballot per bit of the number narrows the set (rows without a
        // cell carry the number L, which no other row has)
        const uint32_t kbits = (uint32_t)(key >= 0 ? key : L);
        uint64_t same = ~0ull;
        for (int bit = 0; bit < nbits; ++bit) {
            const bool set = (kbits >> bit) & 1u;
            const uint64_t bal = __ballot(set);
            same &= set ? bal : ~bal;
        }
        const int lower = __popcll(same & ((1ull << lane) - 1ull));        // earlier rows of this wavefront in the same cell
        uint32_t base = 0;
        for (int turn = 0; turn < kRankRows / 64; ++turn) {
            if (wave == turn && key >= 0 && lower == 0) base = atomicAdd(&cnt[key], (uint32_t)__popcll(same));
            __syncthreads();
        }
        base = __shfl(base, (int)__builtin_ctzll(same));                   // a lane is in its own set: never empty
        if (key >= 0) {
            if (slot) slot[i] = list_base[key] + (int64_t)(base + lower);
            if (order) order[batch_base[key] + (int64_t)(base + lower)] = (int32_t)i;
            if (order_cell) order_cell[batch_base[key] + (int64_t)(base + lower)] = make_int2((int)i, key);
        } else if (i < end && slot) {
            slot[i] = -1;
        }
    }
}

__global__ __launch_bounds__(256) void k_copy_lists(ListStore from, ListStore to) {
    const int l = blockIdx.x;
    const int64_t size = from.list_size[l];
    if (size == 0) return;
    const int64_t src = from.list_off[l], dst = to.list_off[l];
    const int words = from.words;
    const int64_t nblk = (size + 63) / 64;
    const int64_t total_words = nblk * words * 64;
    const uint32_t* s = from.codes + (src >> 6) * words * 64;
    uint32_t* t = to.codes + (dst >> 6) * words * 64;
    for (int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x; e < total_words; e += (int64_t)gridDim.y * 256)
        t[e] = s[e];
    if (to.head && from.head) {
        const int64_t head_total = nblk * from.head_words * 64;
        const uint32_t* hs = from.head + (src >> 6) * from.head_words * 64;
        uint32_t* ht = to.head + (dst >> 6) * from.head_words * 64;
        for (int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x; e < head_total; e += (int64_t)gridDim.y * 256)
            ht[e] = hs[e];
    }
    for (int64_t e = (int64_t)blockIdx.y * 256 + threadIdx.x; e < size; e += (int64_t)gridDim.y * 256) {
        to.gamma[dst + e] = from.gamma[src + e];
        to.ids[dst + e] = from.ids[src + e];
        if (to.xnorm) to.xnorm[dst + e] = from.xnorm ? from.xnorm[src + e] : 0.f;
    }
}

__global__ __launch_bounds__(256) void k_pack_scatter(const uint8_t* __restrict__ codes,
                                                      const uint16_t* __restrict__ gamma,
                                                      const float* __restrict__ xnorm,
                                                      const int64_t* __restrict__ labels, int64_t label_base,
                                                      const int64_t* __restrict__ slot, int64_t n, int d,
                                                      int b, ListStore store) {
    const int words = store.words;
    const int64_t item = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (item >= n * words) return;
    const int64_t row = item / words;
    const int w = (int)(item % words);
    const int64_t s = slot[row];
    if (s < 0) return;
    const uint8_t* c = codes + row * d;
    uint32_t word = 0;
    for (int j = (32 * w) / b; j < d; ++j) {        // coordinate j occupies bits [j*b, j*b + b)
        const int sh = j * b - 32 * w;
        if (sh >= 32) break;
        const uint32_t code = c[j];
        word |= sh >= 0 ? (code << sh) : (code >> (-sh));
    }
    store.codes[((s >> 6) * words + w) * 64 + (s & 63)] = word;
    if (store.head && w < store.head_words) {      // word w of the top-bit plane: coordinate j at bits [j*beta, j*beta + beta)
        const int beta = b - store.head_shift;
        uint32_t hword = 0;
        for (int j = (32 * w) / beta; j < d; ++j) {
            const int sh = j * beta - 32 * w;
            if (sh >= 32) break;
            const uint32_t code = (uint32_t)c[j] >> store.head_shift;
            hword |= sh >= 0 ? (code << sh) : (code >> (-sh));
        }
        store.head[((s >> 6) * store.head_words + w) * 64 + (s & 63)] = hword;
    }
    if (w == 0) {
        store.gamma[s] = gamma[row];
        store.ids[s] = labels ? labels[row] : label_base + row;
        if (store.xnorm) store.xnorm[s] = xnorm ? xnorm[row] : 0.f;
    }
}

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// ---- k-means ------------------------------------------------------------------------------------

// out[l] = sum of count[l'] over l' < l, for up to 16384 entries, by one workgroup.
__global__ __launch_bounds__(1024) void k_exclusive_scan(const uint32_t* __restrict__ count, int L,
                                                         int64_t* __restrict__ out) {
    __shared__ int64_t part[1024];
    const int per = (L + 1023) / 1024;
    const int lo = threadIdx.x * per < L ? threadIdx.x * per : L;
    const int hi = lo + per < L ? lo + per : L;
    int64_t sum = 0;
    for (int l = lo; l < hi; ++l) sum += count[l];
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {            // inclusive running sum over the 1024 parts
        const int64_t add = threadIdx.x >= o ? part[threadIdx.x - o] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int64_t run = part[threadIdx.x] - sum;
    for (int l = lo; l < hi; ++l) { out[l] = run; run += count[l]; }
}

// Sum of the normalised rows of each cell, in a fixed order: workgroup l walks the rows
// order[base[l] .. base[l] + count[l]) of its cell, wavefront w taking every fourth row from the w-th on,
// a lane the coordinates lane, lane + 64, ...; the four partial sums are then added in the order 0, 1, 2, 3.
// Nothing depends on scheduling, so the same input gives the same bits on every run.  Bound by the latency of
// gathering rows: a wavefront reads its next 64 row numbers together and then eight rows together, and adds up
// their squares without LDS (500,000 x 96 over 4096 cells, ten iterations of training: 6355 -> 6019 us).
//
// GAIN (the last iteration, of which the objective is reported): every row's <x~, c> is added up in double as well.
// From the float32 sums it would carry their rounding, which grows with the rows of a cell and is large beside
// the objective of tight cells (400k x 16 rows in 4 cells: 2.6e-5 of it).
// T: coordinates of a lane.
template <bool GAIN, int T>
__global__ __launch_bounds__(256) void k_kmeans_cell_sums(const float* __restrict__ x, int d,
                                                          const int32_t* __restrict__ order,
                                                          const int64_t* __restrict__ base,
                                                          const uint32_t* __restrict__ count,
                                                          float* __restrict__ sums, int pitch,
                                                          const float* __restrict__ cent, double* __restrict__ gain) {
    __shared__ float part[4][64 * T];
    __shared__ double part_gain[4];                  // (GAIN)
    constexpr int U = 8;
    const int l = blockIdx.x, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int64_t first = base[l];
    const int cnt = (int)count[l];
    float acc[T], c[T];
    double g = 0.0;
#pragma unroll
    for (int t = 0; t < T; ++t) {
        acc[t] = 0.f;
        c[t] = GAIN && lane + 64 * t < d ? cent[(int64_t)l * pitch + lane + 64 * t] : 0.f;
    }
    for (int p64 = wave; p64 < cnt; p64 += 4 * 64) {
        const int mine = order[first + (p64 + 4 * lane < cnt ? p64 + 4 * lane : p64)];      // past the end: a row of the cell
        const int rows = (cnt - p64 + 3) / 4 < 64 ? (cnt - p64 + 3) / 4 : 64;
        for (int r = 0; r < rows; r += U) {
            float v[U][T], n2[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float* row = x + (int64_t)__builtin_amdgcn_readlane(mine, r + u) * d;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const int j = lane + 64 * t;
                    v[u][t] = row[j < d ? j : d - 1];
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                n2[u] = 0.f;
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    if (lane + 64 * t >= d) v[u][t] = 0.f;
                    n2[u] += v[u][t] * v[u][t];
                }
                n2[u] = wave_sum(n2[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (r + u >= rows) break;
                const float nrm = sqrtf(n2[u]);
#pragma unroll
                for (int t = 0; t < T; ++t) {
                    const float e = v[u][t] / nrm;
                    acc[t] += e;
                    if (GAIN) g += (double)e * (double)c[t];
                }
            }
        }
    }
#pragma unroll
    for (int t = 0; t < T; ++t) part[wave][lane + 64 * t] = acc[t];
    __syncthreads();
    for (int j = threadIdx.x; j < d; j += 256) sums[(int64_t)l * pitch + j] = ((part[0][j] + part[1][j]) + part[2][j]) + part[3][j];
    if (GAIN) {
        if (wave == 0) {                             // and -|c|^2 / 2 for each of them
#pragma unroll
            for (int t = 0; t < T; ++t) g -= 0.5 * cnt * ((double)c[t] * (double)c[t]);
        }
        for (int o = 32; o > 0; o >>= 1) g += __shfl_xor(g, o);
        if (lane == 0) part_gain[wave] = g;
        __syncthreads();
        if (threadIdx.x == 0) gain[l] = ((part_gain[0] + part_gain[1]) + part_gain[2]) + part_gain[3];
    }
}

// The bias of a centroid row and the row's split form, by one wavefront; the order of the sum is the same everywhere.
__device__ __forceinline__ void finish_centroid(const float* __restrict__ row, int d, int lane, float* __restrict__ bias,
                                                uint16_t* __restrict__ hi, uint16_t* __restrict__ lo) {
    float n2 = 0.f;
    for (int j = lane; j < d; j += 64) {
        const float v = row[j];
        n2 += v * v;
        _Float16 h, l;
        split_scaled(v, h, l);
        hi[j] = __builtin_bit_cast(uint16_t, h);
        lo[j] = __builtin_bit_cast(uint16_t, l);
    }
    for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
    if (lane == 0) *bias = -0.5f * n2;
}

__global__ __launch_bounds__(64) void k_kmeans_update(float* __restrict__ cent, int pitch,
                                                      const float* __restrict__ sums,
                                                      const uint32_t* __restrict__ counts,
                                                      float* __restrict__ bias, uint16_t* __restrict__ cent_h,
                                                      uint16_t* __restrict__ cent_l, int L, int d) {
    const int l = blockIdx.x, lane = threadIdx.x;
    const int64_t at = (int64_t)l * pitch;
    for (int j = d + lane; j < pitch; j += 64) { cent_h[at + j] = 0; cent_l[at + j] = 0; }    // padding columns
    if (l >= L) {
        for (int j = lane; j < d; j += 64) { cent_h[at + j] = 0; cent_l[at + j] = 0; }
        if (lane == 0) bias[l] = -__builtin_inff();
        return;
    }
    const uint32_t c = counts ? counts[l] : 0u;
    if (c > 0)
        for (int j = lane; j < d; j += 64) cent[at + j] = sums[at + j] / (float)c;            // a lane reads back its own values
    finish_centroid(cent + at, d, lane, bias + l, cent_h + at, cent_l + at);
}

// One workgroup: most iterations have no empty cell and leave after the first look at the counts.
__global__ __launch_bounds__(1024) void k_kmeans_reseed(const float* __restrict__ x, int d, const int32_t* __restrict__ order,
                                                        const int64_t* __restrict__ base, const uint32_t* __restrict__ count,
                                                        int L, float* __restrict__ cent, int pitch, float* __restrict__ bias,
                                                        uint16_t* __restrict__ cent_h, uint16_t* __restrict__ cent_l,
                                                        uint64_t seed, unsigned long long* __restrict__ drawn,
                                                        int* __restrict__ row_count) {
    __shared__ unsigned long long s_big;              // largest count, then smallest cell number
    __shared__ uint32_t s_part[1024];
    __shared__ uint16_t s_empty[kMaxList];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int per = (L + 1023) / 1024, lo = tid * per < L ? tid * per : L, hi = lo + per < L ? lo + per : L;
    if (tid == 0) { s_big = 0; *row_count = 0; }
    uint32_t empty = 0;
    unsigned long long big = 0;
    for (int l = lo; l < hi; ++l) {
        const uint32_t c = count[l];
        empty += c == 0;
        const unsigned long long key = ((unsigned long long)c << 32) | (0xFFFFFFFFu - (uint32_t)l);
        big = key > big ? key : big;
    }
    if (!__syncthreads_or(empty != 0)) return;
    atomicMax(&s_big, big);
    s_part[tid] = empty;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const uint32_t add = tid >= o ? s_part[tid - o] : 0;
        __syncthreads();
        s_part[tid] += add;
        __syncthreads();
    }
    uint32_t at = s_part[tid] - empty;
    for (int l = lo; l < hi; ++l)
        if (count[l] == 0) s_empty[at++] = (uint16_t)l;
    __syncthreads();
    const uint32_t total = s_part[1023];
    const int from = (int)(0xFFFFFFFFu - (uint32_t)(s_big & 0xFFFFFFFFull));
    const uint64_t members = s_big >> 32, before = *drawn;
    if (members == 0) return;                         // no row has a cell (none has a usable norm): the call fails
    __syncthreads();
    if (tid == 0) *drawn = before + total;
    for (uint32_t t = wave; t < total; t += 16) {
        // draw number before + t of splitmix64 started at `seed`
        uint64_t z = seed + (before + t + 1) * 0x9E3779B97F4A7C15ull;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        z ^= z >> 31;
        const float* row = x + (int64_t)order[base[from] + (int64_t)(z % members)] * d;
        const int l = s_empty[t];
        float n2 = 0.f;
        for (int j = lane; j < d; j += 64) { const float v = row[j]; n2 += v * v; }
        for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
        const float nrm = sqrtf(n2);
        float* c = cent + (int64_t)l * pitch;
        for (int j = lane; j < d; j += 64) c[j] = nrm > 0.f ? row[j] / nrm : 0.f;
        finish_centroid(c, d, lane, bias + l, cent_h + (int64_t)l * pitch, cent_l + (int64_t)l * pitch);
    }
}

__global__ __launch_bounds__(64) void k_copy_rows_normalised(const float* __restrict__ x, int d,
                                                             const int64_t* __restrict__ src_row,
                                                             const int32_t* __restrict__ dst,
                                                             float* __restrict__ cent, int pitch) {
    const int lane = threadIdx.x;
    const int64_t row = src_row[blockIdx.x];
    const int l = dst[blockIdx.x];
    float n2 = 0.f;
    for (int j = lane; j < d; j += 64) { const float v = x[row * d + j]; n2 += v * v; }
    for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
    const float nrm = sqrtf(n2);
    for (int j = lane; j < d; j += 64) cent[(int64_t)l * pitch + j] = nrm > 0.f ? x[row * d + j] / nrm : 0.f;
}

// Reconstruction of stored vectors (Section "Adaptive coarse refresh", Refresh self-containedness):
// x^ = c~_l + gamma * Pi^T C[code], rows in list order (list l starts at row out_off[l]), labels likewise.
//
// A contraction [vectors] x [d] . [d] x [d] whose result is written once: 4d bytes a vector against 3 * 2d^2 flop on
// the matrix cores, so it should run at the speed of the stores.  Wavefront t of a workgroup owns the output
// coordinates 32t .. 32t + 31 and keeps its 32 columns of Pi^T (both float16 parts, or float32) in registers for the
// life of the workgroup; the 32 vectors of a tile are de-quantised once by all wavefronts together into LDS (in the same
// form, double buffered: one barrier per tile; the next tile's packed words are in flight meanwhile) and are the row operand, so
// that a lane holds one output coordinate of 16 vectors and every store instruction writes whole 128-byte lines.
// For d <= 64 several tiles share a workgroup (SLABS), which keeps it at 128 threads or more.  Workgroups walk
// contiguous ranges of tiles: one search for the list, then steps.
// A call of 1M x 128, b = 4: 0.91 ms with one thread per output coordinate and float32 multiply-adds, 0.16 ms so; the kernel
// takes 114 us of it (5.2 TB/s read + written), the rest is the wait that ends the call.
//
// F32: the operands are float32 (v_mfma_f32_32x32x2_f32) instead of both float16 parts, for d <= kReconF32.  With few
// terms a sum the split form's own rounding (2^-23 of an operand, the same for every use of a level) is what counts:
// against float64 the split results were up to 1.6 times as far off as float32 multiply-adds at d <= 60, never further
// from 61 on, and closer the longer the sum (d = 128: 7.5e-8 against 1.03e-7).  The price, a call of 1M vectors: d = 32
// 47 -> 59 us, d = 48 80 -> 102 us, d = 60 103 -> 122 us (with one thread per output coordinate 145, 194 and 292 us).
constexpr int kReconF32 = 60;
template <int DP, bool F32>
struct ReconCfg {
    static constexpr int KB = DP / 16, NT = DP / 32, LDH = DP + 8;
    static constexpr int SLABS = NT >= 4 ? 1 : (NT == 1 ? 4 : 2);
    static constexpr int THREADS = 64 * NT * SLABS;
    static constexpr int VEC = 32 * SLABS;                       // vectors per tile
    static constexpr int LDF = DP + 4;                           // floats per LDS row
    static constexpr int slab_halves = F32 ? 2 * 32 * LDF : 2 * 32 * LDH;         // float rows, or hi and lo rows
    static constexpr int buf_halves = SLABS * slab_halves;
    static constexpr size_t lds_bytes = (size_t)2 * buf_halves * 2 + 256 * 8 + 2 * VEC * 4;
};

// A value that kernels before this one wrote and none changes now, read through the scalar cache (the compiler would
// use a vector load, and wait for everything in front of it, because this kernel stores to memory it cannot tell apart).
template <class T>
__device__ __forceinline__ T fixed(const T* p) {
    return *reinterpret_cast<const __attribute__((address_space(4))) T*>(reinterpret_cast<uintptr_t>(p));
}

// NW: words that can hold the 8b bits of eight codes (1 for b = 1, 2, 4; 3 for b = 7; else 2)
// PAST: stores go past the caches, where every wavefront's share of a row is whole pieces of 64 bytes, or of 32 in wide rows: pieces that
// wavefronts share have to meet in a cache.  1M rows, past the caches and not, us: 128 coordinates 143 and 171, 112 141 and 181, 80 103 and 120,
// 256 407 and 486; but 100 206 and 174, 124 238 and 201, 68 186 and 121, 72 168 and 122, 104 190 and 177, 250 578 and 480.  Of 8 coordinates and no
// 16, the time of the latter over the former at 1M and 300,000 rows: 168 1.17 and 0.96, 184 1.17 and 1.04, 200 1.02 and 1.03, 232 1.02 and 1.08, 248
// 1.07 and 1.08.  (One kernel with a branch: 160 245 instead of 231.)
template <int DP, int NW, bool F32, bool PAST>
__global__ __launch_bounds__((ReconCfg<DP, F32>::THREADS)) void k_reconstruct(
    ListStore store, int L, const float* __restrict__ cent, int cent_pitch, const float* __restrict__ pi, const uint16_t* __restrict__ pit_h,
    const uint16_t* __restrict__ pit_l, const float* __restrict__ cb, int d, int b, const int64_t* __restrict__ out_off,
    const int32_t* __restrict__ tile_off, int tiles, float* __restrict__ x_out, int64_t* __restrict__ labels_out) {
    using Cfg = ReconCfg<DP, F32>;
    constexpr int KB = Cfg::KB, LDH = Cfg::LDH, LDF = Cfg::LDF, VEC = Cfg::VEC, T = Cfg::THREADS;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint16_t* stage = reinterpret_cast<uint16_t*>(lds_raw);                       // [2][SLABS][hi, lo][32][LDH], or floats [2][SLABS][32][LDF]
    // [2^b] hi | lo << 16, or the float; PAIR (b = 1, 2, 4): [2^2b] both parts of two levels, (hi pair, lo pair)
    constexpr bool PAIR = NW == 1 && !F32;
    uint32_t* tab = reinterpret_cast<uint32_t*>(stage + 2 * Cfg::buf_halves);
    float* gam = reinterpret_cast<float*>(tab + 512);                             // [2][VEC] norms (split form: * 2^-20)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, jl = lane & 31;
    const int col = 32 * (wave % Cfg::NT) + jl, my_slab = wave / Cfg::NT;
    const int words = store.words;
    const uint32_t mask = (1u << b) - 1u;

    // the wavefront's columns of Pi^T: split form, or (F32) element 4g + i of a lane is Pi[8g + 4*half + i][col]
    half8 bh[F32 ? 1 : KB], bl[F32 ? 1 : KB];
    float bf[F32 ? DP / 2 : 1];
    if constexpr (F32) {
#pragma unroll
        for (int e = 0; e < DP / 2; ++e) bf[e] = pi[(8 * (e / 4) + 4 * half + e % 4) * DP + col];
    } else {
#pragma unroll
        for (int kb = 0; kb < KB; ++kb) {
            bh[kb] = *reinterpret_cast<const half8*>(pit_h + (size_t)col * DP + 16 * kb + 8 * half);
            bl[kb] = *reinterpret_cast<const half8*>(pit_l + (size_t)col * DP + 16 * kb + 8 * half);
        }
    }
    for (int e = tid; e < (PAIR ? 1 << 2 * b : (int)mask + 1); e += T) {
        if constexpr (PAIR) {
            _Float16 h0, l0, h1, l1;
            split_scaled(cb[e & mask], h0, l0);
            split_scaled(cb[e >> b], h1, l1);
            reinterpret_cast<uint2*>(tab)[e] = make_uint2((uint32_t)__builtin_bit_cast(uint16_t, h0) | (uint32_t)__builtin_bit_cast(uint16_t, h1) << 16,
                                                          (uint32_t)__builtin_bit_cast(uint16_t, l0) | (uint32_t)__builtin_bit_cast(uint16_t, l1) << 16);
        } else if constexpr (F32) {
            tab[e] = __float_as_uint(cb[e]);
        } else {
            _Float16 h, l;
            split_scaled(cb[e], h, l);
            tab[e] = (uint32_t)__builtin_bit_cast(uint16_t, h) | ((uint32_t)__builtin_bit_cast(uint16_t, l) << 16);
        }
    }

    // this workgroup's tiles, and the list of the first one
    const int per = (tiles + (int)gridDim.x - 1) / (int)gridDim.x;
    const int t_begin = (int)blockIdx.x * per, t_end = t_begin + per < tiles ? t_begin + per : tiles;
    if (t_begin >= t_end) return;
    int l = 0, hi_l = L;
    while (hi_l - l > 1) {
        const int mid = (l + hi_l) >> 1;
        if (tile_off[mid] <= t_begin) l = mid; else hi_l = mid;
    }

    // A tile has VEC * (DP / 8) groups of eight coordinates, two per thread: group tid + p*T is vector (group % 32) of
    // slab group / 32 / (DP/8), coordinates 8*chunk ..; its 8b bits start at bit 8*b*chunk and lie in at most three words.
    // (A word index past the row's end is clamped: codes of coordinates past d meet zeros of Pi^T whatever they are.)
    uint32_t w[2][NW];
    uint32_t next_gam = 0;
    int64_t next_id = 0;
    float next_c = 0.f;
    auto fetch = [&](int l, int n_l, int64_t base, int v0) {
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int e = tid + p * T, v = v0 + 32 * ((e >> 5) / (DP / 8)) + (e & 31), chunk = (e >> 5) % (DP / 8);
            const int64_t slot = base + (v < n_l ? v : n_l - 1);
            const int w0 = (8 * b * chunk) >> 5;
            const uint32_t* wp = store.codes + (slot >> 6) * (int64_t)words * 64 + (slot & 63);
#pragma unroll
            for (int i = 0; i < NW; ++i) w[p][i] = wp[(w0 + i < words ? w0 + i : words - 1) * 64];
        }
        const int v = v0 + (tid < VEC ? tid : VEC - 1);
        const int64_t slot = base + (v < n_l ? v : n_l - 1);
        next_gam = store.gamma[slot];
        next_id = store.ids[slot];
        next_c = cent[(int64_t)l * cent_pitch + col];
    };
    while (t_begin >= fixed(tile_off + l + 1)) ++l;          // lists without vectors have no tile
    int n_l = fixed(store.list_size + l), v0 = (t_begin - fixed(tile_off + l)) * VEC;
    int64_t base = fixed(store.list_off + l), row_l = fixed(out_off + l);
    int tile_end = fixed(tile_off + l + 1);
    fetch(l, n_l, base, v0);

    constexpr float kUnscale = F32 ? 1.f : 1.f / (kSplitScale * kSplitScale);
    int buf = 0;
    __syncthreads();                                 // the table is written
    for (int tile = t_begin; tile < t_end; ++tile, buf ^= 1) {
        const int64_t row0 = row_l + v0;
        uint16_t* st = stage + buf * Cfg::buf_halves;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            const int grp = tid + p * T, slab = (grp >> 5) / (DP / 8), chunk = (grp >> 5) % (DP / 8);
            const int sh = (8 * b * chunk) & 31;
            if constexpr (PAIR) {
                // (hi, lo) of one pair and of the next become (hi, hi) and (lo, lo) by an exchange: four registers in a row to store
                const uint32_t codes = w[p][0] >> sh, both = (1u << 2 * b) - 1u;
                uint32_t r[8];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const uint2 v = reinterpret_cast<const uint2*>(tab)[(codes >> (2 * b * t)) & both];
                    r[2 * t] = v.x;
                    r[2 * t + 1] = v.y;
                }
#pragma unroll
                for (int t = 0; t < 8; t += 4) asm("v_swap_b32 %0, %1" : "+v"(r[t + 1]), "+v"(r[t + 2]));
                uint16_t* row = st + slab * Cfg::slab_halves + (grp & 31) * LDH + 8 * chunk;
                *reinterpret_cast<uint4*>(row) = make_uint4(r[0], r[1], r[4], r[5]);
                *reinterpret_cast<uint4*>(row + 32 * LDH) = make_uint4(r[2], r[3], r[6], r[7]);
                continue;
            }
            uint64_t bits = ((NW > 1 ? (uint64_t)w[p][NW > 1 ? 1 : 0] << 32 : 0ull) | w[p][0]) >> sh;
            if (NW > 2 && sh) bits |= (uint64_t)w[p][NW - 1] << (64 - sh);
            uint32_t e[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) e[t] = tab[(uint32_t)(bits >> (t * b)) & mask];
            if constexpr (F32) {
                uint32_t* row = reinterpret_cast<uint32_t*>(st + slab * Cfg::slab_halves) + (grp & 31) * LDF + 8 * chunk;
                *reinterpret_cast<uint4*>(row) = make_uint4(e[0], e[1], e[2], e[3]);
                *reinterpret_cast<uint4*>(row + 4) = make_uint4(e[4], e[5], e[6], e[7]);
            } else {
                uint32_t hv[4], lv[4];
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    hv[t] = (e[2 * t] & 0xFFFFu) | (e[2 * t + 1] << 16);
                    lv[t] = (e[2 * t] >> 16) | (e[2 * t + 1] & 0xFFFF0000u);
                }
                uint16_t* row = st + slab * Cfg::slab_halves + (grp & 31) * LDH + 8 * chunk;
                *reinterpret_cast<uint4*>(row) = make_uint4(hv[0], hv[1], hv[2], hv[3]);
                *reinterpret_cast<uint4*>(row + 32 * LDH) = make_uint4(lv[0], lv[1], lv[2], lv[3]);
            }
        }
        if (tid < VEC) gam[buf * VEC + tid] = kUnscale * __half2float(__ushort_as_half((uint16_t)next_gam));
        const __amdgpu_buffer_rsrc_t lab = __builtin_amdgcn_make_buffer_rsrc(labels_out + (labels_out ? row0 : 0), 0,
                                                                              labels_out ? min(n_l - v0, VEC) * 8 : 0, 0x00020000);
        typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uint2v, next_id), lab, tid * 8, 0, 0);   // past the end: dropped
        const float c = next_c;
        const int cur_left = n_l - v0 - 32 * my_slab;
        v0 += VEC;
        if (tile + 1 == tile_end) {
            if (tile + 1 < t_end) {
                do ++l; while (tile + 1 >= fixed(tile_off + l + 1));
                n_l = fixed(store.list_size + l);
                base = fixed(store.list_off + l);
                row_l = fixed(out_off + l);
                tile_end = fixed(tile_off + l + 1);
                v0 = 0;
            } else {
                v0 -= VEC;
            }
        }
        fetch(l, n_l, base, v0);                     // (after the last tile: the same tile again, unused)
        // One barrier per tile: the other buffer, written in the next round, was last read before this barrier.
        __syncthreads();
        floatx16 acc;
        const floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        if constexpr (F32) {
            // (a lane's four floats of a read are the terms 8g + 4*half + i of four products, as in bf)
            const float* a_base = reinterpret_cast<const float*>(st + my_slab * Cfg::slab_halves) + jl * LDF + 4 * half;
#pragma unroll
            for (int g = 0; g < DP / 8; ++g) {
                if (8 * g >= d) break;               // (the same for all: what follows is padding)
                const float4 a = *reinterpret_cast<const float4*>(a_base + 8 * g);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.x, bf[F32 ? 4 * g : 0], g ? acc : zero, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.y, bf[F32 ? 4 * g + 1 : 0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.z, bf[F32 ? 4 * g + 2 : 0], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a.w, bf[F32 ? 4 * g + 3 : 0], acc, 0, 0, 0);
            }
        } else {
            const uint16_t* ah_base = st + my_slab * Cfg::slab_halves + jl * LDH + 8 * half;
            const uint16_t* al_base = ah_base + 32 * LDH;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const half8 ah = *reinterpret_cast<const half8*>(ah_base + 16 * kb);
                const half8 al = *reinterpret_cast<const half8*>(al_base + 16 * kb);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[F32 ? 0 : kb], kb ? acc : zero, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[F32 ? 0 : kb], acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[F32 ? 0 : kb], acc, 0, 0, 0);
            }
        }
        // Stores through a buffer descriptor that ends with the list's rows: rows past the list (and columns past d,
        // sent past any end) are dropped by the address check, so every tile issues the same sixteen stores.  Behind
        // tests they could not be counted, and the wait for the next tile's words, which sit in front of them in the
        // memory queue, would be a wait for the stores as well (0.31 ms at 1M x 128 that way).  The whole offset of a row
        // goes through the address register: the check does not cover the scalar offset.
        // (the descriptor is the same for a wavefront, which has to be said: taken for a lane's own, every store became a loop over the
        // descriptors that the lanes might have: kernel 153 us for 1M x 128, 114 now)
        const uint64_t to = reinterpret_cast<uint64_t>(x_out + (row0 + 32 * my_slab) * (int64_t)d);
        const uint32_t to_lo = __builtin_amdgcn_readfirstlane((uint32_t)to), to_hi = __builtin_amdgcn_readfirstlane((uint32_t)(to >> 32));
        const int to_bytes = __builtin_amdgcn_readfirstlane(min(max(cur_left, 0), 32) * d * 4);
        const __amdgpu_buffer_rsrc_t out = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>((uint64_t)to_hi << 32 | to_lo), 0, to_bytes, 0x00020000);
        // (hidden from the compiler, which would keep the sixteen offsets in registers of their own from tile to tile)
        uint32_t at = col < d ? (uint32_t)(4 * half * d + col) * 4u : 0x40000000u;
        asm volatile("" : "+v"(at));
#pragma unroll
        for (int g = 0; g < 4; ++g) {                // result rows 4g .. 4g+3 of a lane: vectors 8g + 4*half ..
            const float4 gm = *reinterpret_cast<const float4*>(gam + buf * VEC + 32 * my_slab + 8 * g + 4 * half);
            const float gg[4] = {gm.x, gm.y, gm.z, gm.w};
#pragma unroll
            for (int i = 0; i < 4; ++i, at += (uint32_t)d * 4u)
                __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(fmaf(gg[i], acc[4 * g + i], c)), out, at, 0, PAST ? 2 : 0);
            at += (uint32_t)d * 16u;
        }
    }
}

// out_off[l] = vectors in the lists before l; tile_off[l] = tiles of `vec` vectors in them (entry L = all)
__global__ __launch_bounds__(1024) void k_list_prefix(const int32_t* __restrict__ size, int L, int vec,
                                                      int64_t* __restrict__ out_off, int32_t* __restrict__ tile_off) {
    __shared__ int64_t part_n[1024];
    __shared__ int32_t part_t[1024];
    const int per = (L + 1023) / 1024, tid = threadIdx.x;
    const int lo = tid * per < L ? tid * per : L, hi = lo + per < L ? lo + per : L;
    int64_t n = 0;
    int32_t t = 0;
    for (int l = lo; l < hi; ++l) { n += size[l]; t += (size[l] + vec - 1) / vec; }
    part_n[tid] = n;
    part_t[tid] = t;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int64_t an = tid >= o ? part_n[tid - o] : 0;
        const int32_t at = tid >= o ? part_t[tid - o] : 0;
        __syncthreads();
        part_n[tid] += an;
        part_t[tid] += at;
        __syncthreads();
    }
    n = part_n[tid] - n;
    t = part_t[tid] - t;
    for (int l = lo; l < hi; ++l) {
        out_off[l] = n;
        tile_off[l] = t;
        n += size[l];
        t += (size[l] + vec - 1) / vec;
    }
    if (tid == 1023) tile_off[L] = part_t[1023];
}

template <int DP, int NW, bool F32, bool PAST>
hipError_t run_reconstruct_as(const ReconstructArgs& a, int cus, hipStream_t st) {
    using Cfg = ReconCfg<DP, F32>;
    static LdsLimit lim;
    const hipError_t e = lim.ensure(reinterpret_cast<const void*>(k_reconstruct<DP, NW, F32, PAST>), Cfg::lds_bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_list_prefix, dim3(1), dim3(1024), 0, st, a.store.list_size, a.L, Cfg::VEC, a.out_off, a.tile_off);
    int64_t tiles = 0;
    for (int l = 0; l < a.L; ++l) tiles += (a.sizes_host[l] + Cfg::VEC - 1) / Cfg::VEC;
    static std::atomic<int> per_cu{0};               // workgroups a compute unit holds, the same on every device of this kind
    int fit = per_cu.load(std::memory_order_relaxed);
    if (fit == 0) {
        const hipError_t eo = hipOccupancyMaxActiveBlocksPerMultiprocessor(&fit, reinterpret_cast<const void*>(k_reconstruct<DP, NW, F32, PAST>), Cfg::THREADS, Cfg::lds_bytes);
        if (eo != hipSuccess) return eo;
        per_cu.store(fit = std::max(fit, 1), std::memory_order_relaxed);
    }
    const unsigned blocks = (unsigned)std::min<int64_t>(tiles, (int64_t)cus * fit);
    hipLaunchKernelGGL((k_reconstruct<DP, NW, F32, PAST>), dim3(blocks), dim3(Cfg::THREADS), Cfg::lds_bytes, st, a.store, a.L, a.cent, a.cent_pitch, a.pi, a.pit_h,
                       a.pit_l, a.cb, a.d, a.b, (const int64_t*)a.out_off, (const int32_t*)a.tile_off, (int)tiles, a.x_out, a.labels_out);
    return hipGetLastError();
}

template <int DP, int NW, bool F32>
hipError_t run_reconstruct_nw(const ReconstructArgs& a, int cus, hipStream_t st) {
    return a.d % (a.d > 160 ? 8 : 16) == 0 && reinterpret_cast<uintptr_t>(a.x_out) % 64 == 0 ? run_reconstruct_as<DP, NW, F32, true>(a, cus, st)
                                                                           : run_reconstruct_as<DP, NW, F32, false>(a, cus, st);
}

// dst[t] = src[idx[t]] for rows of d floats
__global__ __launch_bounds__(64) void k_gather_rows(const float* __restrict__ src, int d,
                                                    const int64_t* __restrict__ idx, float* __restrict__ dst) {
    const int64_t row = idx[blockIdx.x];
    for (int j = threadIdx.x; j < d; j += 64) dst[(int64_t)blockIdx.x * d + j] = src[row * d + j];
}

__global__ __launch_bounds__(64) void k_normalise_centroids(float* __restrict__ cent, int pitch,
                                                            float* __restrict__ bias, int d) {
    const int l = blockIdx.x, lane = threadIdx.x;
    float n2 = 0.f;
    for (int j = lane; j < d; j += 64) { const float v = cent[(int64_t)l * pitch + j]; n2 += v * v; }
    for (int o = 32; o > 0; o >>= 1) n2 += __shfl_xor(n2, o);
    const float nrm = sqrtf(n2);
    for (int j = lane; j < d; j += 64)
        if (nrm > 0.f) cent[(int64_t)l * pitch + j] /= nrm;
    if (lane == 0) bias[l] = 0.f;
}

// Deterministic: one workgroup, fixed summation order.
__global__ __launch_bounds__(256) void k_inertia(const double* __restrict__ gain, int L, int64_t n, double* out) {
    __shared__ double part[256];
    double s = 0.0;
    for (int l = threadIdx.x; l < L; l += 256) s += gain[l];
    part[threadIdx.x] = s;
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (threadIdx.x < o) part[threadIdx.x] += part[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = (double)n - 2.0 * part[0];
}

template <int DP, bool F32>
hipError_t run_reconstruct_as(const ReconstructArgs& a, int cus, hipStream_t st) {
    if (a.b == 1 || a.b == 2 || a.b == 4) return run_reconstruct_nw<DP, 1, F32>(a, cus, st);
    if (a.b == 7) return run_reconstruct_nw<DP, 3, F32>(a, cus, st);
    return run_reconstruct_nw<DP, 2, F32>(a, cus, st);
}

template <int DP>
hipError_t run_reconstruct(const ReconstructArgs& a, int cus, hipStream_t st) {
    if constexpr (DP <= kReconF32) return run_reconstruct_as<DP, true>(a, cus, st);
    else if constexpr (DP - 32 < kReconF32) return a.d <= kReconF32 ? run_reconstruct_as<DP, true>(a, cus, st) : run_reconstruct_as<DP, false>(a, cus, st);
    else return run_reconstruct_as<DP, false>(a, cus, st);
}

}  // namespace

hipError_t launch_segment_hist(const int32_t* assign, int64_t n, int64_t seg_len, int nseg, int L,
                               uint32_t* seg_hist, hipStream_t st) {
    hipLaunchKernelGGL(k_segment_hist, dim3(nseg), dim3(1024), (size_t)L * 4, st, assign, n, seg_len, L, seg_hist);
    return hipGetLastError();
}

hipError_t launch_segment_scan(uint32_t* seg_hist, int nseg, int L, uint32_t* batch_count, const int* flag, int* flag_out, hipStream_t st) {
    if (nseg > kMaxSegments) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_segment_scan, dim3((L + 15) / 16), dim3(1024), 0, st, seg_hist, nseg, L, batch_count, flag, flag_out);
    return hipGetLastError();
}

hipError_t launch_stable_rank(const int32_t* assign, int64_t n, int64_t seg_len, int nseg, int L,
                              const uint32_t* seg_hist, const int64_t* list_base, int64_t* slot,
                              const int64_t* batch_base, int32_t* order, int2* order_cell, const int32_t* new_size, int32_t* list_size, hipStream_t st) {
    hipLaunchKernelGGL(k_stable_rank, dim3(nseg), dim3(kRankRows), (size_t)L * 4, st, assign, n, seg_len, L,
                       seg_hist, list_base, slot, batch_base, order, order_cell, new_size, list_size);
    return hipGetLastError();
}

hipError_t launch_copy_lists(const ListStore& from, const ListStore& to, int L, hipStream_t st) {
    hipLaunchKernelGGL(k_copy_lists, dim3(L, 8), dim3(256), 0, st, from, to);
    return hipGetLastError();
}

hipError_t launch_pack_scatter(const uint8_t* codes, const uint16_t* gamma, const float* xnorm, const int64_t* labels,
                               int64_t label_base, const int64_t* slot, int64_t n, int d, int b,
                               const ListStore& store, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    const int64_t items = n * store.words;
    hipLaunchKernelGGL(k_pack_scatter, dim3((unsigned)((items + 255) / 256)), dim3(256), 0, st, codes, gamma, xnorm,
                       labels, label_base, slot, n, d, b, store);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st) {
    if (n <= 0) return hipSuccess;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3((unsigned)blocks), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_exclusive_scan(const uint32_t* count, int L, int64_t* out, hipStream_t st) {
    if (L < 1 || L > kMaxList) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_exclusive_scan, dim3(1), dim3(1024), 0, st, count, L, out);
    return hipGetLastError();
}

hipError_t launch_kmeans_cell_sums(const float* x, int d, const int32_t* order, const int64_t* base,
                                   const uint32_t* count, int L, float* sums, int pitch, const float* cent,
                                   double* gain, hipStream_t st) {
    if (d > kMaxD) return hipErrorInvalidValue;
    const auto go = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(L), dim3(256), 0, st, x, d, order, base, count, sums, pitch, cent, gain); };
    switch ((d + 63) / 64) {
        case 1: gain ? go(k_kmeans_cell_sums<true, 1>) : go(k_kmeans_cell_sums<false, 1>); break;
        case 2: gain ? go(k_kmeans_cell_sums<true, 2>) : go(k_kmeans_cell_sums<false, 2>); break;
        case 3: gain ? go(k_kmeans_cell_sums<true, 3>) : go(k_kmeans_cell_sums<false, 3>); break;
        default: gain ? go(k_kmeans_cell_sums<true, 4>) : go(k_kmeans_cell_sums<false, 4>); break;
    }
    return hipGetLastError();
}

hipError_t launch_kmeans_update(float* cent, int pitch, const float* sums, const uint32_t* counts,
                                float* bias, uint16_t* cent_h, uint16_t* cent_l, int L, int Lpad, int d, hipStream_t st) {
    hipLaunchKernelGGL(k_kmeans_update, dim3(Lpad), dim3(64), 0, st, cent, pitch, sums, counts, bias, cent_h, cent_l, L, d);
    return hipGetLastError();
}

hipError_t launch_kmeans_reseed(const float* x, int d, const int32_t* order, const int64_t* base, const uint32_t* count,
                                int L, float* cent, int pitch, float* bias, uint16_t* cent_h, uint16_t* cent_l,
                                uint64_t seed, unsigned long long* drawn, int* row_count, hipStream_t st) {
    if (L < 1 || L > kMaxList) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_kmeans_reseed, dim3(1), dim3(1024), 0, st, x, d, order, base, count, L, cent, pitch, bias, cent_h, cent_l, seed,
                       drawn, row_count);
    return hipGetLastError();
}

hipError_t launch_copy_rows_normalised(const float* x, int d, const int64_t* src_row, const int32_t* dst,
                                       int count, float* cent, int pitch, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_rows_normalised, dim3(count), dim3(64), 0, st, x, d, src_row, dst, cent, pitch);
    return hipGetLastError();
}

hipError_t launch_reconstruct(const ReconstructArgs& a, hipStream_t st) {
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    switch (rot_dp(a.d)) {
        case 32: return run_reconstruct<32>(a, cus, st);
        case 64: return run_reconstruct<64>(a, cus, st);
        case 96: return run_reconstruct<96>(a, cus, st);
        case 128: return run_reconstruct<128>(a, cus, st);
        case 160: return run_reconstruct<160>(a, cus, st);
        case 192: return run_reconstruct<192>(a, cus, st);
        case 224: return run_reconstruct<224>(a, cus, st);
        case 256: return run_reconstruct<256>(a, cus, st);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gather_rows(const float* src, int d, const int64_t* idx, int64_t count, float* dst, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_gather_rows, dim3((unsigned)count), dim3(64), 0, st, src, d, idx, dst);
    return hipGetLastError();
}

hipError_t launch_normalise_centroids(float* cent, int pitch, float* bias, int L, int d, hipStream_t st) {
    hipLaunchKernelGGL(k_normalise_centroids, dim3(L), dim3(64), 0, st, cent, pitch, bias, d);
    return hipGetLastError();
}

hipError_t launch_inertia(const double* gain, int L, int64_t n, double* out, hipStream_t st) {
    hipLaunchKernelGGL(k_inertia, dim3(1), dim3(256), 0, st, gain, L, n, out);
    return hipGetLastError();
}

}  // namespace ivftq
