// Internal launcher declarations shared by the HIP translation units of libivftq.
// Nothing here is part of the public ABI (see include/ivftq.h for that).
#pragma once
#include <cmath>
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "search_plan.h"

namespace ivftq {

constexpr int kSlotsPerBlock = 64;   // vectors interleaved in one storage block (= one wavefront)
constexpr int kRowsPerWG = 128;      // data rows one workgroup of the contraction kernels owns
constexpr int kMaxD = 256;
constexpr int kMaxList = 16384;
constexpr int kMaxK = 2048;
constexpr int kPrefixFactorX2 = 2;   // twice the factor f in: dense prefix >= f * k * T / cap vectors
constexpr int kStreamWorkgroups = 8192;             // workgroups the streaming scan aims to launch at least
constexpr int64_t kStreamSliceBytes = 150ll << 20;  // part of the packed index one slice of a large streaming scan covers
constexpr int kMaxGridCells = 4096;  // entries of the quantiser's uniform-grid index (32 KB of LDS)

// Split float16 form used by the float16 matrix-core kernels: V = 1024*v, hi = fp16(V),
// lo = fp16(V - hi).  hi + lo equals V to about 2^-22 relative; the factor keeps lo in the normal
// float16 range for every |v| > 2.4e-4 (below that lo is at most 6e-8 of v's scale).
constexpr float kSplitScale = 1024.f;

// Raises a kernel's dynamic-LDS limit where a launch needs more than the default.  The attribute belongs
// to a (kernel, device) pair, so what has been set is remembered per device (one object per kernel);
// two threads that race here both set it, which is harmless.
class LdsLimit {
  public:
    hipError_t ensure(const void* kernel, size_t bytes) {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
        if (bytes <= set_[dev].load(std::memory_order_acquire)) return hipSuccess;
        e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
        if (e == hipSuccess) set_[dev].store(bytes, std::memory_order_release);
        return e;
    }

  private:
    static constexpr int kDevices = 64;
    std::atomic<size_t> set_[kDevices] = {};
};

// Workgroups of a kernel that fill the current device (its compute units times what one of them holds), for
// launches whose workgroups take their work from a queue; raises the dynamic-LDS limit as well.  Looked up once per
// (kernel, device) pair like LdsLimit.
class ChipFill {
  public:
    hipError_t get(const void* kernel, int threads, size_t lds, unsigned* wgs, unsigned* compute_units = nullptr) {
        int dev = 0, held = 0, units = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kDevices) return hipErrorInvalidDevice;
        uint64_t known = known_[dev].load(std::memory_order_acquire);
        if (!known) {
            e = limit_.ensure(kernel, lds);
            if (e == hipSuccess) e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&held, kernel, threads, lds);
            if (e == hipSuccess) e = hipDeviceGetAttribute(&units, hipDeviceAttributeMultiprocessorCount, dev);
            if (e != hipSuccess) return e;
            if (held < 1 || units < 1) return hipErrorLaunchOutOfResources;
            known = (uint64_t)units << 32 | (uint32_t)(held * units);
            known_[dev].store(known, std::memory_order_release);
        }
        *wgs = (unsigned)known;
        if (compute_units) *compute_units = (unsigned)(known >> 32);
        return hipSuccess;
    }

  private:
    static constexpr int kDevices = 64;
    LdsLimit limit_;
    std::atomic<uint64_t> known_[kDevices] = {};        // compute units << 32 | workgroups
};

inline int round_up(int v, int m) { return (v + m - 1) / m * m; }
inline int64_t round_up64(int64_t v, int64_t m) { return (v + m - 1) / m * m; }

// Padded dimension used by the coarse-scoring kernel (smallest instantiated size >= d).
int coarse_dp(int d);
// Padded dimension used by the rotation kernel (multiple of 32).
inline int rot_dp(int d) { return round_up(d, 32); }
// 32-bit words of packed codes per vector.
inline int code_words(int b, int d) { return (b * d + 31) / 32; }

// Inverted-list storage as the kernels see it.  Slot s of the pool lives in storage block s/64,
// lane s%64; word w of its code sits at codes[(s/64 * words + w) * 64 + s%64], so a wavefront
// reading word w of 64 neighbouring vectors touches 256 contiguous bytes.
struct ListStore {
    uint32_t* codes;
    uint16_t* gamma;          // float16 bit patterns, one per slot
    int64_t* ids;             // labels, one per slot
    float* xnorm;             // |x| of the raw input row, one per slot; null unless the index keeps a raw metric
    const int64_t* list_off;  // [nlist] first slot of each list (multiple of 64)
    const int32_t* list_size; // [nlist] vectors stored in each list
    int words;
    // Optional second copy of the top (b - head_shift) bits of every code, packed the same way in head_words
    // words per vector (pass 1 of the cascade search reads these instead of the full codes); null = not kept.
    uint32_t* head; int head_words; int head_shift;
};

// ---- contraction kernels (split float16 MFMA) --------------------------------------------------------

// scores[i*ld_scores + c] = <x~_i, cent_c> for every c below ld_scores and, with pi_h, the rotated rows z_i = Pi x~_i.
// x: n x d raw rows (normalised inside; what a row without a usable norm gets are not numbers or zero).
// cent_h / cent_l: split float16 form of the centroid table [Lpad][pitch], zero padded, Lpad % 64 == 0
// (made by launch_split_rows).
struct CoarseArgs {
    const float* x; int64_t n; int d;
    const uint16_t* cent_h; const uint16_t* cent_l; int pitch; int Lpad;      // pitch = rot_dp(d)
    float* scores; int64_t ld_scores;
    const uint16_t* pi_h; const uint16_t* pi_l;   // split float16 form of Pi, [pitch][pitch], zero padded (null: no rotation)
    float* z_out;                                 // [n][pitch]
    uint16_t* zh_out; uint16_t* zl_out;           // optional: split float16 form of z
    float* norm_out;                              // optional: |x_i| of every row, 0 where it is not usable
    uint32_t* clear; int clear_n;                 // words that the launch sets to zero (counters of the kernels after it)
};
hipError_t launch_coarse(const CoarseArgs& a, hipStream_t st);
// assign[i] = argmax_c (<x~_i, cent_c> + bias_c), -1 (and *flag = 1) for a row of zero or non-finite norm, in
// two steps: a screening pass with the hi*hi products alone decides every row whose best score is clearly
// ahead, the rest (listed in row_list, counted in *row_count, which the caller clears) is redone with all three
// products.  row_list
// and row_key are scratch arrays of n entries.  part (may be null): scratch of part_entries x 3 floats; with it the
// rows of a last, partly filled round of workgroups and those of a short batch are shared by up to kScreenMaxShares workgroups.
// bias may be null (all zero); the centroids' norms must not exceed 1.
constexpr int kScreenMaxShares = 16;
struct ScreenArgs {
    const float* x; int64_t n; int d;
    const uint16_t* cent_h; const uint16_t* cent_l; int cent_pitch;
    const float* bias; int L; int Lpad;
    int32_t* assign; int* flag; int32_t* row_list; unsigned long long* row_key; int* row_count; float* part; int64_t part_entries;
};
hipError_t launch_coarse_screened(const ScreenArgs& a, hipStream_t st);
// hi[i], lo[i] = split float16 form of src[i]
hipError_t launch_split_rows(const float* src, int64_t count, uint16_t* hi, uint16_t* lo, hipStream_t st);
// hi[c][r], lo[c][r] = split float16 form of src[r][c] (n x n)
hipError_t launch_split_transposed(const float* src, int n, uint16_t* hi, uint16_t* lo, hipStream_t st);

// Pure-MFMA calibration loop: `blocks` workgroups of 4 wavefronts, each wavefront issues 32*iters
// v_mfma_f32_32x32x16_f16.  operands: 4096*8 float16 values (any finite bits); out: blocks*256 floats.
hipError_t launch_mfma_peak(const uint16_t* operands, float* out, int blocks, int iters, hipStream_t st);

// Rotation family.  pi_h/pi_l: split form of Pi, [DP][DP] zero padded, DP = rot_dp(d).
// mode 0: residual -> rotate -> quantise -> pack into the list store at slot[row]
// mode 1: same, but write unpacked codes / fp16 norms to flat arrays (any may be null)
// q_grid: the quantiser's uniform-grid index (host_math.h), q_cells entries of (boundary, index bits).
// order_cell (mode 0): position p of the batch in list order holds row order_cell[p].x, which belongs to list
// order_cell[p].y and goes to slot list_base[l] + p - batch_base[l] (neighbouring lanes store to neighbouring
// slots, and neither the cell nor the slot of a row has to be fetched by row number).  Mode 1 takes the
// rows in input order and reads assign[row].
struct EncodeArgs {
    const float* x; int64_t n; int d; int b;
    const float* cent; int cent_pitch;
    const uint16_t* pi_h; const uint16_t* pi_l;   // split float16 form of Pi, [DP][DP]
    const float2* q_grid; int q_cells; float q_scale, q_offset;
    const int32_t* assign;
    // mode 0
    const int2* order_cell; const int64_t* list_base; const int64_t* batch_base;
    ListStore store; const int64_t* labels; int64_t label_base;
    // mode 1
    uint8_t* codes_flat; uint16_t* gamma_flat;
};

hipError_t launch_encode(int mode, const EncodeArgs& a, hipStream_t st);

// ---- list bookkeeping -------------------------------------------------------------------------

constexpr int kRankRows = 1024;        // rows that a workgroup of the stable counting sort ranks at a time
constexpr int kMaxSegments = 512;      // segments of a batch: the workgroups of 1024 threads that the chip holds (1024 of 512 threads:
                                       // training on 500,000 x 96 5838 -> 5933 us, 10M x 96 built and searched the same)

// seg_hist[s*L + l] = number of rows of segment s assigned to list l (rows with assign < 0 skipped)
hipError_t launch_segment_hist(const int32_t* assign, int64_t n, int64_t seg_len, int nseg, int L,
                               uint32_t* seg_hist, hipStream_t st);
// in place: seg_hist[s][l] <- sum_{s'<s} seg_hist[s'][l];  batch_count[l] <- column total
// (batch_count may be host memory; flag, may be null: a word copied to flag_out)
hipError_t launch_segment_scan(uint32_t* seg_hist, int nseg, int L, uint32_t* batch_count, const int* flag, int* flag_out, hipStream_t st);
// slot[i] = list_base[l] + (rank of row i among the batch rows of list l, in input order); slot and
// list_base may be null when only the order is wanted.
// order (may be null): the batch's rows grouped by list, lists ascending, input order inside a list:
// order[batch_base[l] + rank] = i, with batch_base the exclusive running sum of the batch's rows per list.
// order_cell (may be null): the same order with the list beside the row, order_cell[...] = (i, l).
// new_size (may be null): list_size[l] = new_size[l].
hipError_t launch_stable_rank(const int32_t* assign, int64_t n, int64_t seg_len, int nseg, int L,
                              const uint32_t* seg_hist, const int64_t* list_base, int64_t* slot,
                              const int64_t* batch_base, int32_t* order, int2* order_cell,
                              const int32_t* new_size, int32_t* list_size, hipStream_t st);
// pack already-quantised rows (codes: n x d bytes, one bin number each) into their storage slots
// xnorm (may be null): raw norms of the rows, stored when the store keeps them
hipError_t launch_pack_scatter(const uint8_t* codes, const uint16_t* gamma, const float* xnorm, const int64_t* labels,
                               int64_t label_base, const int64_t* slot, int64_t n, int d, int b,
                               const ListStore& store, hipStream_t st);
// copy every list from one pool layout to another (same words per vector)
hipError_t launch_copy_lists(const ListStore& from, const ListStore& to, int L, hipStream_t st);
hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t st);

// x_out[out_off[l] + v] = cent_l + gamma * Pi^T C[code] for vector v of list l (rows of d floats, list order),
// labels_out (may be null) the stored labels in the same order.  pi: float32 [DP][DP], DP = rot_dp(d), zero padded;
// pit_h / pit_l: split float16 form of Pi^T.  out_off (L entries) and tile_off (L + 1) are scratch, filled by the call; sizes_host:
// the list sizes as the host knows them.
struct ReconstructArgs {
    ListStore store; int L; const int32_t* sizes_host;
    const float* cent; int cent_pitch;
    const float* pi; const uint16_t* pit_h; const uint16_t* pit_l;
    const float* cb; int d; int b;
    int64_t* out_off; int32_t* tile_off;
    float* x_out; int64_t* labels_out;
};
hipError_t launch_reconstruct(const ReconstructArgs& a, hipStream_t st);
// dst[t] = src[idx[t]], rows of d floats
hipError_t launch_gather_rows(const float* src, int d, const int64_t* idx, int64_t count, float* dst, hipStream_t st);

// ---- k-means pieces ---------------------------------------------------------------------------

// out[l] = sum of count[l'] over l' < l (L <= kMaxList)
hipError_t launch_exclusive_scan(const uint32_t* count, int L, int64_t* out, hipStream_t st);
// sums[l][j] = sum of x~_ij over the rows order[base[l] .. base[l] + count[l]) of cell l, added in a fixed
// order (bit-reproducible); rows are normalised on the fly.  gain (may be null): gain[l] = sum over the same rows of
// <x~_i, cent[l]> - |cent[l]|^2 / 2, the cell's share of the sum of best scores, added in double.
hipError_t launch_kmeans_cell_sums(const float* x, int d, const int32_t* order, const int64_t* base,
                                   const uint32_t* count, int L, float* sums, int pitch, const float* cent,
                                   double* gain, hipStream_t st);
// cent[l] = sums[l]/counts[l] for non-empty cells; bias[l] = -|cent_l|^2/2 (padding rows: bias -inf); cent_h / cent_l:
// the split float16 form of the new rows.  count may be null (every cell counts as empty: bias and split form only).
hipError_t launch_kmeans_update(float* cent, int pitch, const float* sums, const uint32_t* counts,
                                float* bias, uint16_t* cent_h, uint16_t* cent_l, int L, int Lpad, int d, hipStream_t st);
// Every empty cell becomes a copy of a random member of the largest cell (the first of them, when several are as
// large): the t-th one, in ascending order, of the member that draw *drawn + t of the splitmix64 sequence of `seed`
// picks; *drawn is then advanced.  order / base / count as above.  Also clears *row_count.
hipError_t launch_kmeans_reseed(const float* x, int d, const int32_t* order, const int64_t* base, const uint32_t* count,
                                int L, float* cent, int pitch, float* bias, uint16_t* cent_h, uint16_t* cent_l,
                                uint64_t seed, unsigned long long* drawn, int* row_count, hipStream_t st);
// cent[dst[t]] = normalised row src_row[t] of x
hipError_t launch_copy_rows_normalised(const float* x, int d, const int64_t* src_row, const int32_t* dst,
                                       int count, float* cent, int pitch, hipStream_t st);
// normalise centroid rows in place; bias <- 0 for real rows
hipError_t launch_normalise_centroids(float* cent, int pitch, float* bias, int L, int d, hipStream_t st);
// *out = n - 2 * sum of gain[l], added in a fixed order
hipError_t launch_inertia(const double* gain, int L, int64_t n, double* out, hipStream_t st);

// ---- search -----------------------------------------------------------------------------------

// cand_off[q*(np+1) + p] = sum_{p'<p} list_size[probe[q][p']]
// first (may be null): first[q] = shortest probe prefix (>= 1 cell) holding at least
// max(k, 2*k*T/cap) vectors, T the query's candidate total; np if there is none.  With `first`, cand_cnt[q],
// gate[0], redo_cnt[q] and redo_done[q] (each may be null) are set to zero: the counters the batched
// scan, its merge and the exact redo add to; and with `rank`, rank[q*np+p] is how many pairs were in the bucket of pair (q, p) before it
// (bucket_cnt counts them; see PairTable).
struct CandOffsetArgs {
    const int32_t* list_size; int32_t* cand_off;
    int k; int cap; int32_t* first;
    int32_t* cand_cnt; int32_t* gate; int32_t* redo_cnt; int32_t* redo_done;
    uint32_t* bucket_cnt; int32_t* rank; int L;
};
constexpr int kSelTake = 192;                   // most winners that the workgroup selection's short cut, which alone reads block maxima, is for
constexpr int64_t kBlockMaximaRow = 8192;       // candidates of a typical row, besides k * k, from which a small streaming call leaves block maxima
// Where the block maxima of a query's probe p begin when `col` candidates precede it.  Every probe has one place more than
// the 64-column groups its candidates touch at most, so that its blocks, counted from its first candidate, fit.
__host__ __device__ constexpr int block_index(int col, int p) { return (col >> 6) + p; }
// scores[q*m_stride + cand_off[q][p] + i] = coarse[q][p] + gamma_i * sum_j z_qj * C[code_ij]
struct ListScanArgs {
    const float* z; int z_pitch; int d;
    const float* cb;
    const int32_t* probe; const float* coarse; const int32_t* cand_off; int np;
    ListStore store;
    float* scores; int64_t m_stride;
    int metric; const float* qnorm;
    // blk_max[q*blk_stride + block_index(cand_off[q][p], p) + b] = order-preserving key of the best score of block b (64
    // vectors) of probe p (null: not wanted)
    uint32_t* blk_max; int64_t blk_stride;
    // Exact redo (gate not null): instead of all queries the entries [gate_begin, gate_begin + gate_count) of the
    // gate[0] queries listed in gate[1..] are scanned.  A query's scores that reach
    // thresh[q*thresh_stride], less the rounding between the arithmetic of the threshold and this one, go, redo_cnt[q] of them in any order, to the
    // first half of one of gate_rows score rows, their columns (cand_off[q][p] + i) to its second half; half a row has to
    // hold every candidate.  redo_done[q] counts the workgroups that have finished their share; the last one writes the k best, by (score
    // desc, label asc), to the query's result row, as values of the metric.
    const int32_t* gate; int gate_begin, gate_count, gate_rows;      // gate_rows: at least gate_count or kRedoWorkgroups (redo_window)
    const float* thresh; int thresh_stride; float slack; int32_t* redo_cnt; int32_t* redo_done;      // slack: the rounding of a sum, per unit of the stored norm
    int k; const int64_t* ids;
    float* out_vals; int64_t* out_i64;
};
constexpr int kRedoThreads = 512;      // of each of the kRedoWorkgroups workgroups
// blocks_per_query: workgroups per query (0 = one per probe), each walking its share of the probes; slices:
// workgroups that share every list.  (Neither matters for a redo.)
hipError_t launch_list_scan(const ListScanArgs& a, int b, int64_t q_count, int blocks_per_query, int slices, hipStream_t st);
// The largest of three values in one instruction; what is no number has no part in it.  Written as one because the compiler quiets every operand of a
// float maximum whose bits it knows nothing of first, an operation a value.
__device__ __forceinline__ float max3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// metric 0: the score is the estimate s^ of <q~, x~> itself.  Raw metrics (the store keeps |x|, qnorm[q] = |q|):
// the scan writes a key that ranks like the metric and whatever writes a call's results turns the selected keys into values:
//   metric 1 (inner product): key = |x| s^,                 value = |q| key            (descending)
//   metric 2 (squared L2):    key = 2 |x| |q| s^ - |x|^2,   value = |q|^2 - key        (ascending; missing: +inf)
__device__ __forceinline__ float metric_key(int metric, float s, float xn, float qn) {
    return metric == 1 ? xn * s : fmaf(2.f * xn * qn, s, -xn * xn);
}
// the factor from a difference of scores to the difference of their keys
__device__ __forceinline__ float metric_scale(int metric, float xn, float qn) { return metric == 1 ? xn : 2.f * xn * qn; }
// An upper bound of metric_key over scores of at most s and lengths in [x_min, x_max].  The inner product key is
// linear in the length; the distance key x (2 |q| s - x) has its one maximum at x = |q| s.  The rounding of a
// key is at most a few units in the last place of its two terms.
__device__ __forceinline__ float metric_key_bound(int metric, float s, float x_min, float x_max, float qn) {
    if (metric == 1) return (s >= 0.f ? x_max : x_min) * s;
    const float x = fminf(fmaxf(qn * s, x_min), x_max);
    return fmaf(2.f * x * qn, s, -x * x) + 0x1p-20f * (x * x + fabsf(2.f * x * qn * s));
}
// (a missing result's key is -inf: it stays so as an inner product, also for a query without a usable norm, whose qn is 0,
// and becomes +inf as a distance)
__device__ __forceinline__ float metric_value(int metric, float key, float qn) {
    if (metric == 1) return key > -__builtin_inff() ? qn * key : -__builtin_inff();
    return qn * qn - key;
}
// Per row: the k largest of m values, sorted by (value desc, label asc).
// mode 0 (probe selection): m = m_fixed for every row, label = column; writes int32 labels.
// mode 1 (results): row q has m = cand_off[q][np] values; column -> (probe p, position) -> label
//                   ids[list_off[probe[q][p]] + position]; writes int64 labels.
struct SelectArgs {
    const float* vals; int64_t stride; int64_t rows; int k;
    int m_fixed;
    const int32_t* cand_off; const int32_t* probe; int np;
    const int32_t* p_limit;   // mode 1: row q only has the candidates of probes p < p_limit[q] (null = all)
    const int64_t* list_off; const int64_t* ids;
    float* out_vals; int32_t* out_i32; int64_t* out_i64;
    int m_bound;      // mode 1: host-side upper bound of any row's length (0 = unknown); picks the kernel
    const uint32_t* blk_max; int64_t blk_stride;      // mode 1: as the scan left them (null: not there)
    int metric; const float* qnorm;                   // mode 1: the values are ranking keys, written as values of the metric
    // mode 0: what follows from the probes just selected (cand.cand_off null: nothing)
    CandOffsetArgs cand;
};
hipError_t launch_select(int mode, const SelectArgs& a, hipStream_t st);

// Exact re-ranking: out = the k candidates of each query with the largest <q~, x~> computed from raw
// rows (x: n_rows x d, addressed by label), ordered by (score desc, label asc), repeats dropped.
struct RerankArgs {
    const float* q; const float* x; int64_t n_rows; int d;
    const int64_t* cand; int r; int k;
    float* out_scores; int64_t* out_ids;
};
hipError_t launch_rerank(const RerankArgs& a, int64_t nq, hipStream_t st);

// Pass 2 of the cascade search: the candidates of each query (slot numbers, -1 = none) are scored
// with the full codes, score = coarse term of the candidate's list + gamma * sum_j z_j cb[code_j],
// and the k best by (score desc, label asc) are written out.
struct CascadeArgs {
    const float* z; int z_pitch; int d; int b;
    const float* cb;                       // 2^b levels
    const int32_t* probe; const float* coarse; int np;     // [nq][np]
    ListStore store;
    const int64_t* ids;                    // label of a slot
    const int64_t* cand; int n_keep; int k;
    float* out_scores; int64_t* out_ids;
};
hipError_t launch_cascade_rescore(const CascadeArgs& a, int64_t nq, hipStream_t st);

// ---- query-batched scan ------------------------------------------------------------------------

// Whether the batched scan covers this (d, b); otherwise the streaming scan is used.
bool batch_covers(int d, int b);
// Panel width of the batched scan for rows of d coordinates: the padded width of the rotated queries (a multiple
// of 32), at least 64, except that 193 ... 208 coordinates take 13 blocks of 16 rather than 14 (d = 200: a
// fourteenth less to de-quantise and multiply).
constexpr int batch_dp(int d) { return (d > 192 && d <= 208) ? 208 : d <= 64 ? 64 : (d + 31) / 32 * 32; }
// Row tiles of 32 queries that a wavefront of the threshold pass holds in registers: up to four, as many as about fit beside their
// accumulators and a slab's words.  Not all of them fit: of 256 registers, 192 coordinates spill 9 to 17, 208 with 2 and 4 bits 16 and 13
// (with 3, 5 and 8, which have two row tiles, none), 224 with 3, 5 and 8 and 256 with 8 bits 4 to 9, and raw metrics, which keep the
// range of the lengths too, up to 26 from 160 coordinates on.  With 208 coordinates of 4 bits one operand is read back in every
// slab; two row tiles, without spills, are slower all the same (10,000 queries at 10M x 200: pass 794 us instead of 766).
constexpr int batch_query_tiles(int dp, int b) {
    const int kb = dp / 16, words = kb * (b == 2 || b == 4 ? 1 : 2);
    return 4 * (4 * kb + 16) + 2 * words <= 180 ? 4 : 3 * 4 * kb + words <= 180 ? 3 : 2;
}
constexpr int batch_tile(int d, int b) { return 32 * batch_query_tiles(batch_dp(d), b); }

// The (query, probe) pairs bucketed by list: bucket l holds the pairs (q, p < first[q]) of list l (the dense pass),
// bucket L + l the pairs (q, p >= first[q]) (the threshold pass).  pairs[pair_off[b] ...] holds the count[b] flat pair
// numbers q*np + p of bucket b.  Its tiles, every tq_near or tq of its queries times the list_parts of its
// list, follow each other in its pass's array (tile_near or tile_late), whose entries name the bucket.
// Each of the kTileQueues queues that the tiles of a pass are dealt out to has a counter.
constexpr int kPairRecord = 8;       // words of a bucket's record
constexpr int kPairTotals = 32 + 2 * kTileQueues * 32;
struct PairTable {
    // cleared with the coarse scores: [2L] pairs of a bucket, then kPairTotals words: totals (pairs, tiles of the dense pass, of
    // the threshold pass) and from word 32 on the next tiles of either pass, kTileQueues counters a cache line apart
    uint32_t* count; int32_t* totals;
    uint32_t* cursor; int32_t* pair_off;      // [2L] each; cursor is scratch
    // [2L] what a tile of a bucket has to know: its list's vectors, its first tile, its pairs, the first of them, its list's first slot (2 words)
    int32_t* record;
    int32_t* tile_near; int32_t* tile_late; int32_t* pairs;
};
// Whether the probe selection counts the buckets' pairs itself: where they are few, and few a list, for its updates of counters, about five
// in a nanosecond over all of them and 14 ns and more apart on one of them, come on top of it; else they are counted in LDS, in two launches
// that take 10 us and more.  Probe selection and grouping, counted early and not, us: 1000 queries x 16 probes of 1000 cells 18.7 and 26, 256 x 64
// of 4096 21 and 29, 1200 x 16 of 600 24 and 27, 10,000 x 32 of 4096 82 and 86, 4096 x 32 of 1024 51 and 32; by pairs a list, 8 probes of 128
// cells: 16 15 and 17, 32 20.7 and 20.8, 64 26 and 22, 128 41 and 24, 250 64 and 27, where one launch fewer saves the call 4 to 6 more (218 x 65 of 388
// 119 and 125, 240 x 72 of 290 83 and 87).
inline bool pairs_counted_early(int64_t nq, int np, int L) { return nq * np <= std::min<int64_t>(32768, (int64_t)64 * L); }
// rank (may be null): as the probe selection left it, with the counts
hipError_t launch_pair_grouping(const int32_t* probe, const int32_t* first, const int32_t* rank, int64_t nq, int np, int L, const int32_t* list_size, const int64_t* list_off,
                                const TileShape& shape, const PairTable& p, hipStream_t st);

struct BatchScanArgs {
    const uint16_t* zh; const uint16_t* zl; int z_pitch;   // split rotated queries, [nq][z_pitch] halves
    const float* cb;
    PairTable p; int part_len;           // part_len of this pass, as the tiles were made
    const float* coarse;                 // [nq*np] coarse term of each (query, probe)
    const float* thresh; int thresh_stride;   // threshold of query q at thresh[q*thresh_stride]
    ListStore store; int np; int L;
    // threshold mode: cand_score = upper bound of the score (see acc0), cand_slot = slot | probe rank << kCandProbeShift
    float* cand_score; int64_t* cand_slot; int32_t* cand_cnt; int cap;
    float acc0;                          // 2^20 * kappa, added to the threshold pass's accumulators
    // dense mode (the nearest lists): every score goes to scores[q*m_stride + cand_off[q][p] + v]
    int dense; float* scores; int64_t m_stride; const int32_t* cand_off;
    int metric; const float* qnorm;      // scores are ranking keys of a raw metric (metric_key)
};
hipError_t launch_batch_scan(const BatchScanArgs& a, int d, int b, hipStream_t st);
// one bit count each, dp = panel width
hipError_t batch_scan_b2(const BatchScanArgs& a, int dp, hipStream_t st);
hipError_t batch_scan_b3(const BatchScanArgs& a, int dp, hipStream_t st);
hipError_t batch_scan_b4(const BatchScanArgs& a, int dp, hipStream_t st);
hipError_t batch_scan_b5(const BatchScanArgs& a, int dp, hipStream_t st);
hipError_t batch_scan_b8(const BatchScanArgs& a, int dp, hipStream_t st);

constexpr int kCandProbeShift = 48;      // a candidate's probe rank sits above its slot number (slots < 2^48, ranks < 2^12)

// kappa with |sum_j z_j c_j - 2^-20 sum_j fp16(1024 z_j) fp16(1024 c_j)| <= kappa for |z| <= 1 and
// codebook values of magnitude <= cmax in d coordinates (each leading part is within 2^-11 relative
// of its value, Cauchy-Schwarz, |c| <= sqrt(d) cmax), with room for float32 accumulation.
inline float screen_kappa(int d, float cmax) { return (0x1p-10f + 0x1p-16f) * 1.002f * sqrtf((float)d) * cmax; }

struct MergeArgs {
    const float* first_scores; const int64_t* first_ids;     // [nq][k] from the dense pass (float32-accurate scores)
    // candidates of the threshold pass: upper bounds u of the score (true score in [u - 2*kappa*gamma, u])
    const float* cand_score; const int64_t* cand_slot; const int32_t* cand_cnt; int cap;
    float kappa;
    int metric; const float* qnorm;                               // as in BatchScanArgs
    const float* z; int z_pitch; int d; int b; const float* cb;   // rotated queries (float32) and levels, for re-scoring
    const float* coarse; int np;                                  // [nq][np] coarse terms
    ListStore store;
    const int64_t* ids;                                       // labels by slot (null: the slot is the label)
    int k; float* out_scores; int64_t* out_ids;
    int32_t* gate;                                            // [1 + nq]: count (cleared by the caller), then the queries whose candidate list overflowed
};
hipError_t launch_merge(const MergeArgs& a, int64_t nq, hipStream_t st);

}  // namespace ivftq
