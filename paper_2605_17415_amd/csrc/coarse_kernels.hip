// Coarse scoring on the matrix cores: <x~_i, c~_l> for every data row i and every cell l, with
// either a running argmax (encode step "assign to the nearest centroid by maximum inner product",
// Section "Architecture", Indexing) or the full score matrix (search step "coarse term computed
// exactly", Section "Architecture", Search).
//
// Shape of the work: n x d times d x L with small d (96..200) and a result that is never kept
// (argmax) or kept once (scores).  One wavefront owns 32*R data rows for the whole kernel and holds
// them in registers as the right-hand MFMA operand; centroid tiles stream through LDS and are the
// left-hand operand, so that in each 32x32 result a lane holds one data row's scores against 16
// centroids and the argmax over centroids never crosses lanes until the very end.
//
// Arithmetic: both operands are used in split float16 form (split_f16.h) on
// v_mfma_f32_32x32x16_f16 with float32 accumulation, so a score differs from the float32 dot
// product by about 2e-7, well inside the 1e-5 near-tie allowance, at the float16 matrix rate.
#include <type_traits>

#include "kernels.h"
#include "split_f16.h"

namespace ivftq {

namespace {

constexpr int kNT = 2;                       // 32-centroid tiles per LDS stage
constexpr int kTN = kNT * 32;

template <int DP>
struct CoarseCfg {
    static constexpr int KB = DP / 16;
    static constexpr int LDH = DP + 8;       // halves per LDS row: the 16-byte pad keeps b128 reads conflict free
    static constexpr size_t lds_bytes = (size_t)2 * kTN * LDH * sizeof(uint16_t);
};

// LDS rows of k_coarse.  Where a compute unit holds three workgroups only without the padding (208 coordinates), the rows go without it
// and 16-byte piece c of row r lies at c ^ (r / 8 & 1) instead: the pitch is then 8 words past a multiple of 16, so that
// sixteen rows read at one piece fall on all 64 banks, as with the padding.  (10,000 queries x 4096 cells x 200, two workgroups with
// padding 143 us, three without 114.)
template <int DP>
struct ScoresCfg {
    static constexpr size_t kLds = 160 * 1024, bare = (size_t)2 * kTN * DP * sizeof(uint16_t);
    static constexpr bool turned = 3 * CoarseCfg<DP>::lds_bytes > kLds && 3 * bare <= kLds;
    static constexpr int LDH = turned ? DP : CoarseCfg<DP>::LDH;
    static constexpr size_t lds_bytes = turned ? bare : CoarseCfg<DP>::lds_bytes;
    static_assert(!turned || DP % 32 == 16, "bank layout");
    static __device__ __forceinline__ int at(int r, int c) { return r * LDH + (turned ? c ^ ((r >> 3) & 1) : c) * 8; }
};

// stages of a call of k_coarse: the centroid table's, then those of Pi
__host__ __device__ constexpr int coarse_stages(const CoarseArgs& a) { return a.Lpad / kTN + (a.pi_h ? (a.pitch + kTN - 1) / kTN : 0); }

// hi[r][c], lo[r][c] = split float16 form of src[r][c]
__global__ void k_split_rows(const float* __restrict__ src, int64_t count, uint16_t* __restrict__ hi,
                             uint16_t* __restrict__ lo) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    _Float16 h, l;
    split_scaled(src[i], h, l);
    hi[i] = __builtin_bit_cast(uint16_t, h);
    lo[i] = __builtin_bit_cast(uint16_t, l);
}

// hi[c][r], lo[c][r] = split float16 form of src[r][c], n x n
__global__ void k_split_transposed(const float* __restrict__ src, int n, uint16_t* __restrict__ hi, uint16_t* __restrict__ lo) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n * n) return;
    _Float16 h, l;
    split_scaled(src[(i % n) * n + i / n], h, l);
    hi[i] = __builtin_bit_cast(uint16_t, h);
    lo[i] = __builtin_bit_cast(uint16_t, l);
}

// One 32-row tile of normalised data rows as the B operand (split form).  Returns whether the
// row's norm is usable; norm (may be null) receives it, 0 for one that is not.
template <int DP>
__device__ __forceinline__ bool load_rows(const float* __restrict__ x, int64_t row, bool valid, int d, int vec4,
                                          int half, half8 (&bh)[DP / 16], half8 (&bl)[DP / 16], float* norm = nullptr) {
    constexpr int KB = DP / 16;
    float v[KB][8];
    load_row_blocks<KB>(x + (valid ? row : 0) * (int64_t)d, valid, d, vec4, half, v);
    const float n2 = row_norm2<KB>(v);
    const bool good = (n2 > 0.f) && (n2 < __builtin_inff());
    const float inv = good ? 1.f / sqrtf(n2) : 0.f;     // one division per row, then multiplies
    if (norm) *norm = good ? sqrtf(n2) : 0.f;
#pragma unroll
    for (int kb = 0; kb < KB; ++kb)
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            _Float16 h, l;
            split_scaled(v[kb][e] * inv, h, l);
            bh[kb][e] = h;
            bl[kb][e] = l;
        }
    return good;
}

// Scores of every row against every centroid and, with a.pi_h, the rotated rows: to this kernel Pi is a few more
// stages of 64 table rows whose products are stored elsewhere.  (A launch of its own for the rotation cost every search
// 5 us, and 12 to 28 us from 256 queries on, where each of its few workgroups walked all of Pi by itself.)
// Workgroup (x, y) takes the row block x and the stages [y * per_y, y * per_y + per_y) of both tables together.
// R = 32-row tiles per wavefront.  VEC4: rows are read 16 bytes at a time (d % 4 == 0, x 16-byte aligned).
// ACROSS: the data rows are the row operand, so that a lane holds 16 rows' scores against one table row and the 32 lanes of a half
// store 128 bytes in a row; else a lane holds one row's scores and stores 16 bytes at a time, 32 rows apart from lane to lane.
template <int DP, int R, bool VEC4, bool ACROSS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(ScoresCfg<DP>::turned ? 3 : 2))) void k_coarse(CoarseArgs a, int per_y) {
    using Cfg = ScoresCfg<DP>;
    constexpr int KB = DP / 16;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint16_t* th = reinterpret_cast<uint16_t*>(lds_raw);            // [TN][LDH] hi parts of the table's rows
    uint16_t* tl = th + kTN * Cfg::LDH;                               // [TN][LDH] lo parts

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, half = lane >> 5, j = lane & 31;
    const int64_t row0 = ((int64_t)blockIdx.x * 4 + wave) * (32 * R);
    for (int i = (int)((blockIdx.y * gridDim.x + blockIdx.x) * 256) + tid; i < a.clear_n; i += (int)(gridDim.x * gridDim.y * 256)) a.clear[i] = 0u;
    const int cent_stages = a.Lpad / kTN, stages = coarse_stages(a);
    const int s_lo = (int)blockIdx.y * per_y, s_hi = s_lo + per_y < stages ? s_lo + per_y : stages;

    // A stage's rows (hi and lo) travel global memory -> registers while the stage before is multiplied and stored, the first
    // one's while the data rows are read, then registers -> LDS, 16 bytes at a time.  (Up to 128 coordinates: one query 28.9 -> 26.4 us,
    // 16 over 10M x 96 55.3 -> 52.8.  Beyond that the registers cost a wavefront per SIMD, and a stage is read when the one before is done.)
    constexpr bool kAhead = DP <= 128;
    constexpr int kPieces = kTN * (DP / 8), kPer = (kPieces + 255) / 256;
    typedef uint32_t piece __attribute__((ext_vector_type(4)));
    piece pre_h[kAhead ? kPer : 1], pre_l[kAhead ? kPer : 1];      // (a native vector: arrays of uint4 went through scratch memory)
#define IVFTQ_COARSE_FETCH(S)                                                                                    \
    {                                                                                                            \
        const bool rot_ = (S) >= cent_stages;                                                                    \
        const int c0_ = (rot_ ? (S) - cent_stages : (S)) * kTN;                                                  \
        const uint16_t* src_h_ = rot_ ? a.pi_h : a.cent_h;                                                       \
        const uint16_t* src_l_ = rot_ ? a.pi_l : a.cent_l;                                                       \
        const int last_ = (rot_ ? a.pitch : a.Lpad) - 1;      /* Pi has `pitch` rows, not a whole number of stages */ \
        _Pragma("unroll") for (int i = 0; i < kPer; ++i) {                                                       \
            const int e_ = tid + 256 * i < kPieces ? tid + 256 * i : kPieces - 1, r_ = c0_ + e_ / (DP / 8);      \
            const int64_t src_ = (int64_t)(r_ < last_ ? r_ : last_) * a.pitch + e_ % (DP / 8) * 8;               \
            pre_h[i] = *reinterpret_cast<const piece*>(src_h_ + src_);                                           \
            pre_l[i] = *reinterpret_cast<const piece*>(src_l_ + src_);                                           \
        }                                                                                                        \
    }
    if constexpr (kAhead) IVFTQ_COARSE_FETCH(s_lo)

    half8 bh[R][KB], bl[R][KB];
    bool any[R];                         // (whether the tile has a row at all: a few queries leave most tiles without)
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t row = row0 + 32 * r + j;
        any[r] = !kAhead || row0 + 32 * r < a.n;
        if (!any[r]) continue;
        float norm;
        load_rows<DP>(a.x, row, row < a.n, a.d, VEC4 ? 1 : 0, half, bh[r], bl[r], &norm);
        if (a.norm_out && s_lo == 0 && half == 0 && row < a.n) a.norm_out[row] = norm;
    }
    const uint16_t* ah_base = th + Cfg::at(j, half);       // (pieces 2 kb + half of rows j and 32 + j: the same turn)
    const uint16_t* al_base = tl + Cfg::at(j, half);
    constexpr float kUnscale = 1.f / (kSplitScale * kSplitScale);

    for (int s = s_lo; s < s_hi; ++s) {
        const bool rotate = s >= cent_stages;
        const int c0 = (rotate ? s - cent_stages : s) * kTN;
        __syncthreads();
        if constexpr (kAhead) {
#pragma unroll
            for (int i = 0; i < kPer; ++i) {
                const int e = tid + 256 * i;
                if (kPieces % 256 == 0 || e < kPieces) {
                    *reinterpret_cast<piece*>(th + Cfg::at(e / (DP / 8), e % (DP / 8))) = pre_h[i];
                    *reinterpret_cast<piece*>(tl + Cfg::at(e / (DP / 8), e % (DP / 8))) = pre_l[i];
                }
            }
        } else {
            const uint16_t* src_h = rotate ? a.pi_h : a.cent_h;
            const uint16_t* src_l = rotate ? a.pi_l : a.cent_l;
            const int last = (rotate ? a.pitch : a.Lpad) - 1;
            for (int e = tid; e < kPieces; e += 256) {
                const int r = e / (DP / 8), c8 = e % (DP / 8);
                const int64_t src = (int64_t)(c0 + r < last ? c0 + r : last) * a.pitch + c8 * 8;
                *reinterpret_cast<uint4*>(th + Cfg::at(r, c8)) = *reinterpret_cast<const uint4*>(src_h + src);
                *reinterpret_cast<uint4*>(tl + Cfg::at(r, c8)) = *reinterpret_cast<const uint4*>(src_l + src);
            }
        }
        __syncthreads();
        if constexpr (kAhead)
            if (s + 1 < s_hi) IVFTQ_COARSE_FETCH(s + 1)
        if (row0 >= a.n) continue;

        floatx16 acc[R][kNT];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int t = 0; t < kNT; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[r][t][q] = 0.f;
        auto product = [](half8 table, half8 row, floatx16 c) {
            return ACROSS ? __builtin_amdgcn_mfma_f32_32x32x16_f16(row, table, c, 0, 0, 0) : __builtin_amdgcn_mfma_f32_32x32x16_f16(table, row, c, 0, 0, 0);
        };
        auto multiply = [&](auto tiles) {
            constexpr int RR = decltype(tiles)::value;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
#pragma unroll
                for (int t = 0; t < kNT; ++t) {
                    const half8 ah = *reinterpret_cast<const half8*>(ah_base + t * 32 * Cfg::LDH + 16 * kb);
                    const half8 al = *reinterpret_cast<const half8*>(al_base + t * 32 * Cfg::LDH + 16 * kb);
#pragma unroll
                    for (int r = 0; r < RR; ++r) acc[r][t] = product(ah, bh[r][kb], acc[r][t]);
#pragma unroll
                    for (int r = 0; r < RR; ++r) acc[r][t] = product(ah, bl[r][kb], acc[r][t]);
#pragma unroll
                    for (int r = 0; r < RR; ++r) acc[r][t] = product(al, bh[r][kb], acc[r][t]);
                }
            }
        };
        if (R == 1 || any[R - 1]) multiply(std::integral_constant<int, R>{});
        else multiply(std::integral_constant<int, 1>{});

        if constexpr (!ACROSS) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t row = row0 + 32 * r + j;
                if (row >= a.n) continue;
#pragma unroll
                for (int t = 0; t < kNT; ++t)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int c = c0 + t * 32 + 8 * g + 4 * half;
                        const float4 o = make_float4(acc[r][t][4 * g] * kUnscale, acc[r][t][4 * g + 1] * kUnscale,
                                                     acc[r][t][4 * g + 2] * kUnscale, acc[r][t][4 * g + 3] * kUnscale);
                        if (!rotate) {
                            if (c < a.ld_scores) *reinterpret_cast<float4*>(a.scores + row * a.ld_scores + c) = o;
                        } else if (c < a.pitch) {
                            const int64_t at = row * a.pitch + c;
                            *reinterpret_cast<float4*>(a.z_out + at) = o;
                            if (a.zh_out) {
                                const float z[4] = {o.x, o.y, o.z, o.w};
                                uint16_t h[4], l[4];
#pragma unroll
                                for (int e = 0; e < 4; ++e) {
                                    _Float16 hi, lo;
                                    split_scaled(z[e], hi, lo);
                                    h[e] = __builtin_bit_cast(uint16_t, hi);
                                    l[e] = __builtin_bit_cast(uint16_t, lo);
                                }
                                *reinterpret_cast<uint2*>(a.zh_out + at) = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
                                *reinterpret_cast<uint2*>(a.zl_out + at) = make_uint2(l[0] | ((uint32_t)l[1] << 16), l[2] | ((uint32_t)l[3] << 16));
                            }
                        }
                    }
            }
        } else {
            // result row q of a lane: row 8 (q / 4) + 4 half + q % 4 of the tile
            const int width = rotate ? a.pitch : a.ld_scores;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const int64_t rest = a.n - (row0 + 32 * r);
                int left = (rest < 32 ? (int)rest : 32) - 4 * half;            // rows of the tile from this half's first on
#pragma unroll
                for (int t = 0; t < kNT; ++t) {
                    const int c = c0 + t * 32 + j;
                    if (c >= width) continue;
                    const uint32_t own = (uint32_t)(4 * half * width + j);
                    int64_t at = (row0 + 32 * r) * width + c0 + t * 32;        // (the same for all lanes)
                    asm volatile("" : "+s"(at), "+v"(left));     // or what follows for all rows and tiles is worked out ahead and spilled
                    if (!rotate) {
                        float* out = a.scores + at;
#pragma unroll
                        for (int q = 0; q < 16; ++q) {
                            if (8 * (q / 4) >= rest) break;
                            if (8 * (q / 4) + q % 4 < left) out[own] = acc[r][t][q] * kUnscale;
                            out += q % 4 == 3 ? 5 * width : width;
                        }
                        continue;
                    }
#pragma unroll
                    for (int q = 0; q < 16; ++q) {
                        if (8 * (q / 4) >= rest) break;
                        if (8 * (q / 4) + q % 4 < left) {
                            const float o = acc[r][t][q] * kUnscale;
                            (a.z_out + at)[own] = o;
                            if (a.zh_out) {
                                _Float16 hi, lo;
                                split_scaled(o, hi, lo);
                                (a.zh_out + at)[own] = __builtin_bit_cast(uint16_t, hi);
                                (a.zl_out + at)[own] = __builtin_bit_cast(uint16_t, lo);
                            }
                        }
                        at += q % 4 == 3 ? 5 * width : width;
                    }
                }
            }
        }
    }
}

#undef IVFTQ_COARSE_FETCH

// Screening pass of the argmax: only the hi*hi products (one MFMA per block instead of three).  With
// unit vectors the result is off by at most (2^-10 + 2^-22) * sum|a_j b_j| <= 9.8e-4 plus float32
// summation error, so when the best screened score beats the second best by more than twice that, the
// best is the exact argmax as well.  Rows where it does not (and rows without a usable norm) are
// appended to row_list and redone by k_coarse_resolve with all three products; both write assign.
// Per score: best' = max(best, v), second' = med3(best, second, v).
constexpr float kScreenMargin = 2.2e-3f;
constexpr float kScreenNone = -3.0e38f;     // below every score, finite so that tagging its low bits keeps it a number

// 32-centroid tiles per LDS stage of the screening pass (two stages are resident)
template <int DP>
constexpr int screen_nt() { return 2; }

template <int DP>
constexpr size_t screen_lds_bytes(bool bias) {
    return (size_t)2 * screen_nt<DP>() * 32 * (CoarseCfg<DP>::LDH * sizeof(uint16_t) + (bias ? sizeof(float) : 0));
}

// (The scores carry a tag in their low bits and are never NaN: max3 of kernels.h, and the middle of three as the compiler's builtin.)

// The 16 scores of tile position t that a lane holds, four at a time.  The position (t, q) replaces
// the low 6 bits of the float32 pattern (a change below 2^-17 of the score's size), so that maxima and
// medians alone carry the index.  With b the running best and s the running second best, two new
// scores u, w give  s' = max(s, med3(b, u, w)),  b' = max(b, u, w).
#define IVFTQ_SCREEN_TAKE(MASKED)                                                                          \
    _Pragma("unroll") for (int q = 0; q < 16; q += 4) {                                                     \
        _Pragma("unroll") for (int r = 0; r < R; ++r) {                                                     \
            float v[4];                                                                                     \
            _Pragma("unroll") for (int i = 0; i < 4; ++i) {                                                 \
                v[i] = __uint_as_float((__float_as_uint(acc[r][q + i]) & ~63u) | (unsigned)(t * 16 + q + i)); \
                /* columns q..q+3 of a lane are neighbouring centroids 8*(q/4) + 4*half + i */              \
                if (MASKED) v[i] = (c0 + t * 32 + 2 * q + 4 * half + i < L) ? v[i] : kScreenNone;           \
            }                                                                                               \
            const float m0 = __builtin_amdgcn_fmed3f(best[r], v[0], v[1]);                                  \
            const float b1 = max3(best[r], v[0], v[1]);                                                 \
            const float m1 = __builtin_amdgcn_fmed3f(b1, v[2], v[3]);                                       \
            best[r] = max3(b1, v[2], v[3]);                                                             \
            second[r] = max3(second[r], m0, m1);                                                        \
        }                                                                                                   \
    }

// VEC4: rows are read 16 bytes at a time (d % 4 == 0 and x 16-byte aligned); a template parameter so that
// each instantiation carries one loading path only (with both, the loads of the prologue spill).
// BIAS: the argmax is of <x~, c> + bias_c, |c| <= 1 (k-means: c a mean of unit vectors, bias_c = -|c|^2/2).  The
// accumulators of a tile start at 2^20 bias_c; the error of the products is bounded as without it.
template <int DP, int R, bool VEC4, bool BIAS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu((DP <= 128 || R == 1) ? 3 : 2))) void k_coarse_screen(
    const float* __restrict__ x, int64_t n, int d, const uint16_t* __restrict__ cent_h, int cent_pitch,
    const float* __restrict__ bias, int L, int Lpad, int32_t* __restrict__ assign, int32_t* __restrict__ row_list,
    unsigned long long* __restrict__ row_key, int* __restrict__ row_count, float* __restrict__ part, int whole, int shares) {
    using Cfg = CoarseCfg<DP>;
    constexpr int KB = Cfg::KB;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    constexpr int NT = screen_nt<DP>(), TN = NT * 32;
    // The first `whole` row blocks are one workgroup's each.  Every later one is shared by `shares` workgroups: each takes its
    // share of the centroid stages and leaves (best, second best, index) of every row in `part`, where
    // k_coarse_screen_join puts them together.
    const bool split = (int)blockIdx.x >= whole;
    // Eight blocks at a time, share by share: every eighth workgroup runs on the same one of the chip's eight parts, so that the
    // workgroups of a block meet in one L2 cache and its rows are read from memory once.  (Next to each other: 2000 rows x 96
    // over 4096 cells 21.2 us instead of 20.)
    const int n_stages = Lpad / TN;
    int block = (int)blockIdx.x, share = 0, per_share = n_stages;
    if (split) {
        const int rest = block - whole, split_blocks = ((int)gridDim.x - whole) / shares;
        const int eight = rest / (8 * shares) * 8, in_eight = rest - eight * shares, side = split_blocks - eight < 8 ? split_blocks - eight : 8;
        block = whole + eight + in_eight % side;
        share = in_eight / side;
        per_share = (n_stages + shares - 1) / shares;
    }
    const int c_lo = share * per_share * TN < Lpad ? share * per_share * TN : Lpad;
    const int c_hi = c_lo + per_share * TN < Lpad ? c_lo + per_share * TN : Lpad;
    uint16_t* th = reinterpret_cast<uint16_t*>(lds_raw);            // [2][TN][LDH] hi parts of the centroids
    float* s_bias = reinterpret_cast<float*>(th + 2 * TN * Cfg::LDH);   // [2][TN] 2^20 bias (BIAS only)
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, half = lane >> 5, j = lane & 31;
    const int64_t row0 = ((int64_t)block * 4 + wave) * (32 * R);

    half8 bh[R][KB];
    bool good[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int64_t row = row0 + 32 * r + j;
        half8 unused[KB];
        good[r] = load_rows<DP>(x, row, row < n, d, VEC4 ? 1 : 0, half, bh[r], unused);
        __builtin_amdgcn_sched_barrier(0);          // one tile's float32 values at a time in registers
    }
    float best[R], second[R];
    int best_c0[R];
#pragma unroll
    for (int r = 0; r < R; ++r) { best[r] = kScreenNone; second[r] = kScreenNone; best_c0[r] = 0; }
    // Stage s+1 travels global memory -> registers while stage s is multiplied, then registers -> the
    // other LDS buffer; one barrier per stage.
    constexpr int kChunks = TN * (DP / 8);                          // 16-byte pieces of one stage
    constexpr int kPer = (kChunks + 255) / 256;
    uint4 pre[kPer];
    float pre_bias = 0.f;
#define IVFTQ_SCREEN_FETCH(C0)                                                                     \
    if (BIAS) pre_bias = bias[(C0) + (tid & (TN - 1)) < Lpad ? (C0) + (tid & (TN - 1)) : Lpad - 1];  \
    _Pragma("unroll") for (int i = 0; i < kPer; ++i) {                                              \
        int e = tid + 256 * i;                                                                      \
        e = e < kChunks ? e : kChunks - 1;                                                          \
        const int r = e / (DP / 8), c8 = e % (DP / 8);                                              \
        const int c = (C0) + r < Lpad ? (C0) + r : Lpad - 1; /* a stage may reach past the padded rows */ \
        pre[i] = *reinterpret_cast<const uint4*>(cent_h + (int64_t)c * cent_pitch + c8 * 8);        \
    }
#define IVFTQ_SCREEN_STORE(STAGE)                                                                  \
    if (BIAS && tid < TN) s_bias[(STAGE) * TN + tid] = pre_bias * (kSplitScale * kSplitScale);       \
    _Pragma("unroll") for (int i = 0; i < kPer; ++i) {                                              \
        const int e = tid + 256 * i;                                                                \
        if (kChunks % 256 == 0 || e < kChunks)                                                      \
            *reinterpret_cast<uint4*>(th + (STAGE) * (TN * Cfg::LDH) + (e / (DP / 8)) * Cfg::LDH + (e % (DP / 8)) * 8) = pre[i]; \
    }
    IVFTQ_SCREEN_FETCH(c_lo)
    IVFTQ_SCREEN_STORE(0)
    __syncthreads();
    int stage = 0;
    for (int c0 = c_lo; c0 < c_hi; c0 += TN, stage ^= 1) {
        IVFTQ_SCREEN_FETCH(c0 + TN)          // unconditional (indices are clamped): after the last stage it is unused
        const uint16_t* ah_base = th + stage * (TN * Cfg::LDH) + j * Cfg::LDH + 8 * half;
        float prev[R];
#pragma unroll
        for (int r = 0; r < R; ++r) prev[r] = best[r];
        // The row operand of a tile is read from LDS a tile ahead: the reads of tile t+1 are issued
        // after the products of tile t and complete while its scores are taken.
        // (up to 128 coordinates; beyond that the registers do not reach and each block is read as it is used)
        constexpr bool kAhead = KB <= 8;
        half8 ah[kAhead ? KB : 1];
        if (kAhead) {
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) ah[kAhead ? kb : 0] = *reinterpret_cast<const half8*>(ah_base + 16 * kb);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
            floatx16 acc[R];
            if constexpr (BIAS) {
#pragma unroll
                for (int g = 0; g < 4; ++g) {       // accumulator 4g + i of a lane: centroid 8g + 4*half + i of the tile
                    const float4 b4 = *reinterpret_cast<const float4*>(s_bias + stage * TN + t * 32 + 8 * g + 4 * half);
#pragma unroll
                    for (int r = 0; r < R; ++r) {
                        acc[r][4 * g] = b4.x; acc[r][4 * g + 1] = b4.y;
                        acc[r][4 * g + 2] = b4.z; acc[r][4 * g + 3] = b4.w;
                    }
                }
            } else {
#pragma unroll
                for (int r = 0; r < R; ++r)
#pragma unroll
                    for (int q = 0; q < 16; ++q) acc[r][q] = 0.f;
            }
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                const half8 a = kAhead ? ah[kAhead ? kb : 0]
                                       : *reinterpret_cast<const half8*>(ah_base + t * 32 * Cfg::LDH + 16 * kb);
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, bh[r][kb], acc[r], 0, 0, 0);
            }
            if (kAhead && t + 1 < NT) {
#pragma unroll
                for (int kb = 0; kb < KB; ++kb)
                    ah[kAhead ? kb : 0] = *reinterpret_cast<const half8*>(ah_base + (t + 1) * 32 * Cfg::LDH + 16 * kb);
            }
            if (c0 + (t + 1) * 32 <= L) {
                IVFTQ_SCREEN_TAKE(false)
            } else {
                IVFTQ_SCREEN_TAKE(true)
            }
        }
        // which stage the best came from is seen from whether the stage changed it
#pragma unroll
        for (int r = 0; r < R; ++r) best_c0[r] = best[r] != prev[r] ? c0 : best_c0[r];
        IVFTQ_SCREEN_STORE(stage ^ 1)
        __syncthreads();
    }
#undef IVFTQ_SCREEN_FETCH
#undef IVFTQ_SCREEN_STORE
    uint64_t undecided[R];
    int mine = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const unsigned code = __float_as_uint(best[r]) & 63u;
        int idx = best_c0[r] + (int)(code >> 4) * 32 + 8 * (int)((code & 15u) >> 2) + 4 * half + (int)(code & 3u);
        // the other half of the lane pair saw the other centroids of the same row
        const float ob = __shfl_xor(best[r], 32), os = __shfl_xor(second[r], 32);
        const int oi = __shfl_xor(idx, 32);
        const float s2 = fmaxf(fmaxf(second[r], os), fminf(best[r], ob));
        const float b2 = fmaxf(best[r], ob);
        if (ob > best[r]) idx = oi;
        const int64_t row = row0 + 32 * r + j;
        if (split) {
            if (row < n && half == 0) {
                float* pp = part + ((row - (int64_t)whole * (4 * 32 * R)) * shares + share) * 3;
                pp[0] = b2;
                pp[1] = s2;
                pp[2] = __int_as_float(good[r] ? idx : -1 - idx);
            }
            continue;
        }
        const bool own = row < n && half == 0, sure = good[r] && (b2 - s2 > kScreenMargin * kSplitScale * kSplitScale);
        if (own) assign[row] = idx;
        undecided[r] = __ballot(own && !sure);
        mine += __popcll(undecided[r]);
    }
    if (split) return;
    // One update of the list's counter for a workgroup: updates of one word from all over the chip follow each other.  (Encoding without
    // clusters, 300 cells, with one for every 32 rows and now: 65,516 rows x 20 40 us and 28, 50,527 x 32 38 and 28.)
    int* s_cnt = reinterpret_cast<int*>(lds_raw);      // [4] by wavefront, [4] the first position (nobody reads the stages any more)
    if (lane == 0) s_cnt[wave] = mine;
    __syncthreads();
    int at = 0, all = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        const int c = s_cnt[w];
        at += w < wave ? c : 0;
        all += c;
    }
    if (all == 0) return;
    if (tid == 0) s_cnt[4] = atomicAdd(row_count, all);
    __syncthreads();
    at += s_cnt[4];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (undecided[r] >> lane & 1) {
            const int pos = at + __popcll(undecided[r] & ((1ull << lane) - 1ull));
            row_list[pos] = (int32_t)(row0 + 32 * r + j);
            row_key[pos] = 0ull;
        }
        at += __popcll(undecided[r]);
    }
}
#undef IVFTQ_SCREEN_TAKE

// Shares of a row's screening pass put together: the best of the bests, and as second best the largest of
// every share's second best and of the bests that lost; then the same decision as in the kernel itself.  `part` starts
// at the row first_row.
__global__ void k_coarse_screen_join(const float* __restrict__ part, int64_t first_row, int64_t n, int shares, int32_t* __restrict__ assign,
                                     int32_t* __restrict__ row_list, unsigned long long* __restrict__ row_key,
                                     int* __restrict__ row_count) {
    const int64_t at = (int64_t)blockIdx.x * blockDim.x + threadIdx.x, row = first_row + at;
    if (row >= n) return;
    float best = kScreenNone, second = kScreenNone;
    int idx = 0;
    bool good = true;
    for (int y = 0; y < shares; ++y) {
        const float* pp = part + (at * shares + y) * 3;
        const float b = pp[0], s2 = pp[1];
        int i = __float_as_int(pp[2]);
        if (i < 0) { good = false; i = -1 - i; }
        if (b > best) { second = fmaxf(second, best); best = b; idx = i; }
        else second = fmaxf(second, b);
        second = fmaxf(second, s2);
    }
    const bool sure = good && (best - second > kScreenMargin * kSplitScale * kSplitScale);
    assign[row] = idx;
    if (!sure) {
        const int pos = atomicAdd(row_count, 1);
        row_list[pos] = (int32_t)row;
        row_key[pos] = 0ull;
    }
}

// The undecided rows of the screening pass, with all three products.  Workgroup (x, y) walks the row
// blocks x, x + gridDim.x, ... of the list (128 rows each, one tile per wavefront) against the y-th share of
// the centroid stages, so that a short list still spreads over the chip; the shares of a row meet in
// row_key[position] through a 64-bit atomic maximum of (order-preserving score bits, ~index), which keeps
// the smallest index among equal scores like the single-kernel argmax does.  A row without a usable norm
// leaves its key at 0.
// BIAS is a template parameter: tested per score at run time it cost an encode of 11,866 unclustered rows x 58 (589
// cells), most of them undecided, 41.6 us instead of 40.0.
template <int DP, bool VEC4, bool BIAS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_coarse_resolve(
    const float* __restrict__ x, int d, const uint16_t* __restrict__ cent_h,
    const uint16_t* __restrict__ cent_l, int cent_pitch, const float* __restrict__ bias, int L, int Lpad, const int32_t* __restrict__ row_list,
    const int* __restrict__ row_count, unsigned long long* __restrict__ row_key) {
    using Cfg = CoarseCfg<DP>;
    constexpr int KB = Cfg::KB;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    uint16_t* th = reinterpret_cast<uint16_t*>(lds_raw);            // [TN][LDH] hi parts of the centroid tile
    uint16_t* tl = th + kTN * Cfg::LDH;                               // [TN][LDH] lo parts
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63, half = lane >> 5, j = lane & 31;
    const int n = *row_count;
    const int stages = Lpad / kTN, per_y = (stages + (int)gridDim.y - 1) / (int)gridDim.y;
    const int c_lo = (int)blockIdx.y * per_y * kTN;
    const int c_hi = c_lo + per_y * kTN < Lpad ? c_lo + per_y * kTN : Lpad;
    if (c_lo >= c_hi) return;
    const uint16_t* ah_base = th + j * Cfg::LDH + 8 * half;
    const uint16_t* al_base = tl + j * Cfg::LDH + 8 * half;

    for (int64_t rb = blockIdx.x; rb * 128 < n; rb += gridDim.x) {
        const int pos = (int)(rb * 128) + wave * 32 + j;
        half8 bh[KB], bl[KB];
        const bool good = load_rows<DP>(x, pos < n ? (int64_t)row_list[pos] : 0, pos < n, d, VEC4 ? 1 : 0, half, bh, bl);
        float best = -__builtin_inff();
        int best_idx = 0;
        for (int c0 = c_lo; c0 < c_hi; c0 += kTN) {
            __syncthreads();                 // the previous stage (or row block) is no longer read
            for (int e = tid; e < kTN * (DP / 8); e += 256) {
                const int r = e / (DP / 8), c8 = e % (DP / 8);
                const int64_t src = (int64_t)(c0 + r) * cent_pitch + c8 * 8;
                *reinterpret_cast<uint4*>(th + r * Cfg::LDH + c8 * 8) = *reinterpret_cast<const uint4*>(cent_h + src);
                *reinterpret_cast<uint4*>(tl + r * Cfg::LDH + c8 * 8) = *reinterpret_cast<const uint4*>(cent_l + src);
            }
            __syncthreads();
            floatx16 acc[kNT];
#pragma unroll
            for (int t = 0; t < kNT; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) acc[t][q] = 0.f;
#pragma unroll
            for (int kb = 0; kb < KB; ++kb)
#pragma unroll
                for (int t = 0; t < kNT; ++t) {
                    const half8 ah = *reinterpret_cast<const half8*>(ah_base + t * 32 * Cfg::LDH + 16 * kb);
                    const half8 al = *reinterpret_cast<const half8*>(al_base + t * 32 * Cfg::LDH + 16 * kb);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bh[kb], acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ah, bl[kb], acc[t], 0, 0, 0);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(al, bh[kb], acc[t], 0, 0, 0);
                }
            // raw accumulators (the argmax does not depend on the common 2^20 scale), or with a bias true units;
            // ascending c, first maximum wins
#pragma unroll
            for (int t = 0; t < kNT; ++t)
#pragma unroll
                for (int q = 0; q < 16; ++q) {
                    const int c = c0 + t * 32 + 8 * (q / 4) + 4 * half + (q % 4);
                    const float v = BIAS ? fmaf(acc[t][q], 1.f / (kSplitScale * kSplitScale), bias[c]) : acc[t][q];
                    if (c < L && v > best) { best = v; best_idx = c; }
                }
        }
        const float ob = __shfl_xor(best, 32);
        const int oi = __shfl_xor(best_idx, 32);
        if (ob > best || (ob == best && oi < best_idx)) { best = ob; best_idx = oi; }
        if (pos < n && half == 0 && good) {
            const unsigned u = __float_as_uint(best);
            const unsigned mono = (u & 0x80000000u) ? ~u : (u | 0x80000000u);
            atomicMax(row_key + pos, ((unsigned long long)mono << 32) | (unsigned long long)(0xFFFFFFFFu - (unsigned)best_idx));
        }
    }
}

__global__ void k_coarse_resolve_write(const int32_t* __restrict__ row_list, const int* __restrict__ row_count,
                                       const unsigned long long* __restrict__ row_key, int32_t* __restrict__ assign,
                                       int* __restrict__ flag) {
    const int n = *row_count;
    for (int pos = blockIdx.x * blockDim.x + threadIdx.x; pos < n; pos += gridDim.x * blockDim.x) {
        const unsigned long long key = row_key[pos];
        assign[row_list[pos]] = key ? (int32_t)(0xFFFFFFFFu - (unsigned)(key & 0xFFFFFFFFull)) : -1;
        if (!key) atomicOr(flag, 1);
    }
}

// RS = 32-row tiles per wavefront of the screening kernel
template <int DP, int RS, bool VEC4, bool BIAS>
hipError_t run_screened_as(const ScreenArgs& a, hipStream_t st) {
    static LdsLimit lim_resolve;
    static ChipFill fill;
    const size_t lds_screen = screen_lds_bytes<DP>(BIAS);
    const size_t lds = (size_t)2 * kTN * CoarseCfg<DP>::LDH * sizeof(uint16_t);
    hipError_t e = lim_resolve.ensure(reinterpret_cast<const void*>(k_coarse_resolve<DP, VEC4, BIAS>), lds);
    if (e != hipSuccess) return e;
    constexpr int kBlockRows = 4 * 32 * RS;
    unsigned held = 0, units = 0;
    e = fill.get(reinterpret_cast<const void*>(k_coarse_screen<DP, RS, VEC4, BIAS>), 256, lds_screen, &held, &units);
    if (e != hipSuccess) return e;
    // Rounds of row blocks that fill the chip are a workgroup a block.  The blocks of a last round, or of a short batch, are
    // shared out over the centroid stages where that is faster, given room for the partial results.  Measured (32 to
    // 256 coordinates, 256 to 4096 centroids, 500 to 300,000 rows, 1 to 16 shares): with m workgroups a compute unit a
    // stage takes as m, one alone as 1.7 (up to 64 coordinates, of which a unit holds four, one to three as 1.9, 2.4 and 3.2); reading and
    // splitting the rows of each takes 4 more, and the joining launch 3 us, about 350 / DP of them.  A finer split has to be
    // cheaper by 3 %.  Assignment, us, whole and in the shares that this chooses: 4096 centroids, 262,147 rows x 200 (one block of 1025 left
    // over) 659 and 558 (16); 50,000 x 200 188 and 122 (5); 100,000 x 32 65 and 59 (3); 65,000 x 96 91 and 67 (2); 2000 x 96 73 and 20 (16).  On
    // 420 sizes it is within 3 % of a fixed rule (powers of 2 up to 1024 workgroups, no split from 262,144 rows on) or faster.
    const int64_t blocks = (a.n + kBlockRows - 1) / kBlockRows;
    const int64_t rest = blocks % held, n_stages = a.Lpad / (screen_nt<DP>() * 32);
    int shares = 1;
    auto cost = [&](int64_t s) {           // in tenths of a stage
        const int64_t m = (rest * s + units - 1) / units;
        const int64_t stage = DP <= 64 ? (m <= 1 ? 19 : m == 2 ? 24 : m == 3 ? 32 : 10 * m) : m <= 1 ? 17 : 10 * m;
        return stage * ((n_stages + s - 1) / s) + 40 * m + (s > 1 ? 3500 / DP : 0);
    };
    if (a.part && rest) {
        int64_t least = cost(1);
        for (int s = 2; s <= kScreenMaxShares && 2 * s <= n_stages && rest * kBlockRows * s <= a.part_entries; ++s)
            if (100 * cost(s) < 97 * least) { least = cost(s); shares = s; }
    }
    const int64_t whole = shares > 1 ? blocks - rest : blocks, first = whole * kBlockRows;
    hipLaunchKernelGGL((k_coarse_screen<DP, RS, VEC4, BIAS>), dim3((unsigned)(whole + (blocks - whole) * shares)), dim3(256), lds_screen, st, a.x, a.n, a.d,
                       a.cent_h, a.cent_pitch, a.bias, a.L, a.Lpad, a.assign, a.row_list, a.row_key, a.row_count, a.part, (int)whole, shares);
    if (first < a.n)
        hipLaunchKernelGGL(k_coarse_screen_join, dim3((unsigned)((a.n - first + 255) / 256)), dim3(256), 0, st, (const float*)a.part, first, a.n, shares,
                           a.assign, a.row_list, a.row_key, a.row_count);
    // the undecided rows: about four centroid stages per workgroup, at most 512 x 16 workgroups
    const int stages = a.Lpad / kTN;
    const int ysplit = std::min(16, (stages + 3) / 4);
    const int64_t row_blocks = (a.n + 127) / 128;
    const dim3 grid_r((unsigned)std::min<int64_t>(row_blocks, 512), (unsigned)ysplit);
    hipLaunchKernelGGL((k_coarse_resolve<DP, VEC4, BIAS>), grid_r, dim3(256), lds, st, a.x, a.d, a.cent_h, a.cent_l, a.cent_pitch, a.bias, a.L, a.Lpad,
                       (const int32_t*)a.row_list, (const int*)a.row_count, a.row_key);
    hipLaunchKernelGGL(k_coarse_resolve_write, dim3((unsigned)std::min<int64_t>((a.n + 255) / 256, 256)), dim3(256), 0, st,
                       (const int32_t*)a.row_list, (const int*)a.row_count, (const unsigned long long*)a.row_key, a.assign, a.flag);
    return hipGetLastError();
}

template <int DP, int RS>
hipError_t run_screened(const ScreenArgs& a, hipStream_t st) {
    const bool vec4 = (a.d % 4 == 0) && (reinterpret_cast<uintptr_t>(a.x) % 16 == 0);
    if (a.bias) return vec4 ? run_screened_as<DP, RS, true, true>(a, st) : run_screened_as<DP, RS, false, true>(a, st);
    return vec4 ? run_screened_as<DP, RS, true, false>(a, st) : run_screened_as<DP, RS, false, false>(a, st);
}

template <int DP, int R, bool VEC4, bool ACROSS>
hipError_t run_as(const CoarseArgs& a, hipStream_t st) {
    static ChipFill fill;
    constexpr size_t lds = ScoresCfg<DP>::lds_bytes;
    unsigned held = 0;
    const hipError_t e = fill.get(reinterpret_cast<const void*>(k_coarse<DP, R, VEC4, ACROSS>), 256, lds, &held);
    if (e != hipSuccess) return e;
    const int64_t blocks = (a.n + 4 * 32 * R - 1) / (4 * 32 * R);
    // Every (row, table row) result is independent, so the stages of a row block can be shared out as one likes.  A
    // workgroup of s stages takes about s + 1 stage times (its rows are read, normalised and split first), and
    // the launch as many rounds of them as it has workgroups for the places on the chip: the split with the fewest stage
    // times in all, the finer one of equals.
    const int stages = coarse_stages(a);
    int per_y = 1;
    int64_t least = INT64_MAX;
    for (int s = 1; s <= stages; ++s) {
        const int64_t wgs = blocks * ((stages + s - 1) / s), cost = (wgs + held - 1) / held * (s + 1);
        if (cost < least) { least = cost; per_y = s; }
    }
    hipLaunchKernelGGL((k_coarse<DP, R, VEC4, ACROSS>), dim3((unsigned)blocks, (unsigned)((stages + per_y - 1) / per_y)), dim3(256), lds, st, a, per_y);
    return hipGetLastError();
}

template <int DP, int R>
hipError_t run(const CoarseArgs& a, hipStream_t st) {
    const bool vec4 = (a.d % 4 == 0) && (reinterpret_cast<uintptr_t>(a.x) % 16 == 0);
    // Stores of whole lines are four times as many instructions, most of them for rows that a small call does not have, and pay
    // where there are many scores to store.  Coarse scores and 8 probes, without against with them, us: 4096 queries x 1024 cells x 32 23.8
    // and 25.3, x 96 27.4 and 28.8; 10,000 x 1024 x 32 37.0 and 38.5, x 96 43.6 and 41.5; 30,000 x 1024 x 32 69 and 67; 4096 x 4096 x 96
    // 50.7 and 49.3; 10,000 x 4096 x 96 98.9 and 95.6; 30,000 x 4096 x 96 299 and 276, x 200 565 and 396.
    if (a.n * a.Lpad > (int64_t)8 << 20) return vec4 ? run_as<DP, R, true, true>(a, st) : run_as<DP, R, false, true>(a, st);
    return vec4 ? run_as<DP, R, true, false>(a, st) : run_as<DP, R, false, false>(a, st);
}

// Calibration of the float16 matrix pipe: nothing but v_mfma_f32_32x32x16_f16 on operands held in
// registers, four independent accumulators per wavefront, two wavefronts per SIMD.  What this
// reaches with random operand bits is the rate the contraction kernels can be compared with: the
// chip lowers its clock under the switching activity of real data, so it is below the nominal peak.
__global__ __launch_bounds__(256) void k_mfma_peak(const half8* __restrict__ src, float* __restrict__ out, int iters) {
    half8 a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        a[i] = src[(threadIdx.x * 16 + i) & 4095];
        b[i] = src[(threadIdx.x * 16 + 8 + i) & 4095];
    }
    floatx16 acc[4];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[c][q] = 0.f;
    for (int it = 0; it < iters; ++it) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int c = 0; c < 4; ++c) acc[c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[(i + c) & 7], b[i], acc[c], 0, 0, 0);
    }
    float s = 0.f;
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int q = 0; q < 16; ++q) s += acc[c][q];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = s;
}

}  // namespace

hipError_t launch_mfma_peak(const uint16_t* operands, float* out, int blocks, int iters, hipStream_t st) {
    hipLaunchKernelGGL(k_mfma_peak, dim3(blocks), dim3(256), 0, st, reinterpret_cast<const half8*>(operands), out, iters);
    return hipGetLastError();
}

int coarse_dp(int d) {
    static const int sizes[] = {32, 64, 96, 128, 160, 192, 208, 224, 256};
    for (int s : sizes)
        if (d <= s) return s;
    return -1;
}

hipError_t launch_split_rows(const float* src, int64_t count, uint16_t* hi, uint16_t* lo, hipStream_t st) {
    if (count <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_split_rows, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, st, src, count, hi, lo);
    return hipGetLastError();
}

hipError_t launch_split_transposed(const float* src, int n, uint16_t* hi, uint16_t* lo, hipStream_t st) {
    hipLaunchKernelGGL(k_split_transposed, dim3((unsigned)((n * n + 255) / 256)), dim3(256), 0, st, src, n, hi, lo);
    return hipGetLastError();
}

hipError_t launch_coarse_screened(const ScreenArgs& a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    switch (coarse_dp(a.d)) {
#define IVFTQ_CASE(DPV) \
    case DPV: return run_screened<DPV, 2>(a, st);
        IVFTQ_CASE(32) IVFTQ_CASE(64) IVFTQ_CASE(96) IVFTQ_CASE(128) IVFTQ_CASE(160)
        IVFTQ_CASE(192) IVFTQ_CASE(208) IVFTQ_CASE(224) IVFTQ_CASE(256)
#undef IVFTQ_CASE
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_coarse(const CoarseArgs& a, hipStream_t st) {
    if (a.n <= 0) return hipSuccess;
    switch (coarse_dp(a.d)) {
#define IVFTQ_CASE(DPV, RV) \
    case DPV: return run<DPV, RV>(a, st);
        IVFTQ_CASE(32, 2) IVFTQ_CASE(64, 2) IVFTQ_CASE(96, 2) IVFTQ_CASE(128, 2) IVFTQ_CASE(160, 1)
        IVFTQ_CASE(192, 1) IVFTQ_CASE(208, 1) IVFTQ_CASE(224, 1) IVFTQ_CASE(256, 1)
#undef IVFTQ_CASE
        default: return hipErrorInvalidValue;
    }
}

}  // namespace ivftq
