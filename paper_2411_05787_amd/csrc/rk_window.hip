// Prefill-side initialisation of the small cache from an observation window: rk_window_select.
//
// The W queries of the last prompt tokens vote for the rows of the full cache (Section 2.2
// "Prefilling stage": the scores of the last prompt token; Section 3 and Appendix A.1 "Baseline
// Settings": the last few tokens of the prompt, the observation window).  Per query head,
//   votes[j] = sum_i softmax_{j' <= p_i}(scale <q_i, k_j'>)[j],  p_i = len - W + i  (causal),
// then the selection of rk_topk_select runs on the votes.
//
// Only K is read, twice:
//   pass 1  window_lse_kernel     maximum and sum of every (query, head) column, split over
//                                 workgroups like the decode kernels; pass 2, or window_lse_merge_kernel,
//                                 folds the partial (max, sum) pairs
//   pass 2  window_vote_kernel    the same stream again: normalised scores, summed over the
//                                 window's queries on the lanes, stored once per (head, row)
// Storing the raw scores of every query instead (one pass) would write and re-read
// W * Hq * len * 4 bytes: more than the second pass over K from W = 8 on at the usual shapes.
//
// Per tile of 16 to 64 rows the scores of all columns come from the matrix cores
// (v_mfma_f32_16x16x32_bf16, K rows as the 16-row operand straight from global memory in
// operand layout; the queries, 16 columns at a time, from LDS).  Column c = i * Gp + gi: query
// i of the window, head gi of the GQA group, Gp = G rounded up to a power of two so that a lane
// keeps the same head in every block of 16 columns and the sum over the window is a per-lane
// sum over blocks plus log2(16 / Gp) cross-lane steps.
#include "rk_internal.h"
#include <cfloat>
#include <cmath>
#include <type_traits>
#include "rk_device.h"

namespace rk {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

struct WindowParams {
    const uint16_t* q;                 // bf16 [B, W, Hq, 128]
    const uint16_t* k; int64_t s_b, s_h; int32_t cap;
    const int32_t* seq_lens; int32_t max_rows;
    int32_t W, G, gp_shift;            // Gp = 1 << gp_shift
    int32_t ncb;                       // blocks of 16 columns
    int32_t nch, wg_rows, Hq, Hkv;     // workgroups per (sequence, KV head); rows a workgroup takes per step
    float scale2;                      // |scale| x log2 e, not 0: scores, maxima and exponents are to base 2
    uint32_t q_sign;                   // 0x80008000 where the scale is negative: the queries take its sign
    float* part;                       // fp32 [B*Hkv][nch][ncb*16][2]  (max, sum) per workgroup and column
    float* lse;                        // fp32 [B*Hkv][ncb*16][2]       maximum and 1 / sum of every column (0, 0: nobody votes in it)
    float* votes; int64_t v_stride; int32_t v_vec;
    const int32_t* pred; int32_t pred_val;
};

constexpr int kQStride = kD + 8;       // bf16 elements between columns in LDS: 272 bytes, conflict-free 16-byte reads

__device__ __forceinline__ int window_workgroups(const WindowParams& p, int n_rows) {
    return max(1, min(p.nch, (n_rows + p.wg_rows - 1) / p.wg_rows));
}

// Last row that column `col` may see (-1: the column does not exist).
__device__ __forceinline__ int column_limit(const WindowParams& p, int col, int n) {
    const int i = col >> p.gp_shift, gi = col & ((1 << p.gp_shift) - 1);
    const int pos = n - p.W + i;
    return (i < p.W && gi < p.G && pos >= 0) ? pos : -1;
}

// The window's queries of KV head g go to LDS, one column per (query, head), zero where none, 16 pieces of
// 16 bytes per column.  In two parts, request and store, so that the request can go out ahead of the first rows'
// (memory answers a wavefront in the order of its requests) and nobody waits for rows to have the queries:
// the request holds the first kQHeld pieces of a thread (128 columns in all), a wider window's rest is
// copied by the store.
constexpr int kQHeld = 4;
__device__ __forceinline__ uint4 query_piece(const WindowParams& p, int b, int g, int n, int x) {
    const int col = x >> 4, piece = x & 15;
    if (column_limit(p, col, n) < 0) return make_uint4(0, 0, 0, 0);
    const int i = col >> p.gp_shift, gi = col & ((1 << p.gp_shift) - 1);
    return *reinterpret_cast<const uint4*>(p.q + (((int64_t)b * p.W + i) * p.Hq + (int64_t)g * p.G + gi) * kD + piece * 8);
}
template <int NT>
__device__ __forceinline__ void request_queries(const WindowParams& p, int b, int g, int n, uint4 (&held)[kQHeld]) {
#pragma unroll
    for (int u = 0; u < kQHeld; ++u) held[u] = query_piece(p, b, g, n, u * NT + threadIdx.x);
}
template <int NT>
__device__ __forceinline__ void store_queries(const WindowParams& p, int b, int g, int n, int ncol, const uint4 (&held)[kQHeld],
                                              uint16_t* sQ) {
    auto put = [&](int x, const uint4 u) {
        *reinterpret_cast<uint4*>(sQ + (x >> 4) * kQStride + (x & 15) * 8) = make_uint4(u.x ^ p.q_sign, u.y ^ p.q_sign, u.z ^ p.q_sign, u.w ^ p.q_sign);
    };
#pragma unroll
    for (int u = 0; u < kQHeld; ++u)
        if (u * NT + (int)threadIdx.x < ncol * 16) put(u * NT + threadIdx.x, held[u]);
    for (int x = kQHeld * NT + threadIdx.x; x < ncol * 16; x += NT) put(x, query_piece(p, b, g, n, x));
}

// Rows r .. r + 16 T - 1 of K in operand layout (rows past the end repeat the last row; masked later).
template <int T>
__device__ __forceinline__ void load_k_rows(u32x4 (&dst)[T][4], const uint16_t* kb, int r, int n16, int n) {
#pragma unroll
    for (int t = 0; t < T; ++t) {
        const int row = min(r + t * 16 + n16, n - 1);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            dst[t][kk] = *reinterpret_cast<const u32x4*>(kb + (int64_t)row * kD + kk * 32);
    }
}

// Products of these rows with the 16 columns of block cb: x[t][i] is row r + 16 t + 4 c4 + i of
// column cb * 16 + n16; MASKED: -inf beyond `limit`.  Scores are scale2 times that, and both passes take them
// relative to a maximum M in one rounding, 2^fma(x, scale2, -M): were they rounded before the subtraction in one of the passes and not in the
// other, a column's votes would carry the rounding of its largest score (1.4e-5 at scores of 400).
template <bool MASKED, int T>
__device__ __forceinline__ void block_products(const u32x4 (&k)[T][4], const uint16_t* sQ, int cb, int n16, int c4,
                                               int r, int limit, float (&x)[T][4]) {
    bf16x8 qa[4];
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
        qa[kk] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(sQ + (cb * 16 + n16) * kQStride + (kk * 4 + c4) * 8));
#pragma unroll
    for (int t = 0; t < T; ++t) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, k[t][kk]), qa[kk], acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            x[t][i] = (!MASKED || r + t * 16 + 4 * c4 + i <= limit) ? acc[i] : -INFINITY;
    }
}

// (m, l) <- (m, l) merged with (m2, l2): running max and sum of exponentials relative to it.
__device__ __forceinline__ void merge_ml(float& m, float& l, float m2, float l2) {
    const float M = fmaxf(m, m2);
    const float a = (m == -INFINITY) ? 0.f : fast_exp2(m - M);
    const float c = (m2 == -INFINITY) ? 0.f : fast_exp2(m2 - M);
    l = l * a + l2 * c;
    m = M;
}

extern __shared__ __attribute__((aligned(16))) unsigned char window_lds[];

// Both passes: a wavefront takes 16 T rows at a time and goes through the blocks of columns with them in
// registers, so that a block's queries are read from LDS, and its running state is updated, once per 16 T
// rows; eight wavefronts share one copy of the queries, and two such workgroups per CU (four wavefronts
// per SIMD, up to 128 columns) hide one another's chains; the rows are requested behind the queries and before
// anything waits, so at 32768 rows of 8 KV heads all of K is in flight at once.  The causal masks are worked out only
// for rows that some query does not see.  Bound: the vector instructions of 8 exponentials per 32 x 16 scores from about
// 16 queries on, memory below.  The forms (window_form):
//   T = 4, S = 1  rows enough to give every wavefront of the chip 64; us at 32 heads over 8, 32768 rows, 32 queries, with K
//                 in the last-level cache: 41.7 + 26.7 (32 rows, 4 wavefronts per workgroup, 3 per CU) -> 25.1 + 20.8 (K from
//                 memory: 28.3 + 26.6); the queries requested behind the rows instead of before them: 27.3 + 23.9
//   T = 2, S = 2  up to 32 columns, where a step is short and bound by memory, and up to 128 where the rows would leave the
//                 last round of T = 4 half empty: two sets of 32 rows, each requested again as soon as it is used, 4 wavefronts per workgroup (finer: the last round of a row is not full;
//                 8 wavefronts and 4 sets of 16 rows were 2-3% slower at 33000 to 60000 rows); 0-4% over the form with
//                 masks everywhere, most for K in the last-level cache
//   T = 1, S = 1  few rows: more, shorter wavefronts (3000 rows, 32 queries, the whole case: 45.6 with T = 4, 34.9)
//
// Pass 1.  The running (max, sum) of a lane's column in every block lives in LDS (one float2 per
// lane and block), so that the number of blocks is a run-time value and the register count does
// not grow with the window.
template <bool MASKED, int T, int NT>
__device__ __forceinline__ void lse_rows(const WindowParams& p, const u32x4 (&k)[T][4], const uint16_t* sQ,
                                         float2* sRun, int r, int n, bool first) {
    const int lane = threadIdx.x & 63, n16 = lane & 15, c4 = lane >> 4;
#pragma unroll 1
    for (int cb = 0; cb < p.ncb; ++cb) {
        float x[T][4];
        block_products<MASKED, T>(k, sQ, cb, n16, c4, r, MASKED ? column_limit(p, cb * 16 + n16, n) : 0, x);
        float mx = x[0][0];
#pragma unroll
        for (int e = 1; e < 4 * T; ++e) mx = fmaxf(mx, x[e >> 2][e & 3]);
        const float2 run = first ? make_float2(-INFINITY, 0.f) : sRun[cb * NT + threadIdx.x];
        const float m_new = fmaxf(run.x, mx * p.scale2);
        const float ref = m_new == -INFINITY ? 0.f : m_new;      // nothing seen yet: every term is 2^-inf = 0
        float ps = 0.f;
#pragma unroll
        for (int e = 0; e < 4 * T; ++e) ps += fast_exp2(fmaf(x[e >> 2][e & 3], p.scale2, -ref));
        sRun[cb * NT + threadIdx.x] = make_float2(m_new, run.y * fast_exp2(run.x - ref) + ps);
    }
}

template <int T, int S, int NW>
__global__ __launch_bounds__(NW * 64, 4)
void window_lse_kernel(const WindowParams p) {
    const int ncb = p.ncb, ncol = ncb * 16;
    const int c = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    if (p.pred != nullptr && p.pred[b] != p.pred_val) return;
    const int n = min(max(min(p.seq_lens[b], p.cap), 0), p.max_rows);
    if (n == 0 || c >= window_workgroups(p, n)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n16 = lane & 15, c4 = lane >> 4;
    uint16_t* sQ = reinterpret_cast<uint16_t*>(window_lds);
    float2* sRun = reinterpret_cast<float2*>(window_lds + (size_t)ncol * kQStride * 2);   // [ncb][NW * 64]

    const uint16_t* kb = p.k + (int64_t)b * p.s_b + (int64_t)g * p.s_h + c4 * 8;
    const int step = p.nch * NW * 16 * T, r0 = (c * NW + w) * 16 * T;
    uint4 held[kQHeld];
    u32x4 k[S][T][4];
    request_queries<NW * 64>(p, b, g, n, held);
#pragma unroll
    for (int x = 0; x < S; ++x)
        if (r0 + x * step < n) load_k_rows<T>(k[x], kb, r0 + x * step, n16, n);
    store_queries<NW * 64>(p, b, g, n, ncol, held, sQ);
    __syncthreads();
    auto rows = [&](const u32x4 (&x)[T][4], int r) {
        if (r + 16 * T > n - p.W) lse_rows<true, T, NW * 64>(p, x, sQ, sRun, r, n, r == r0);
        else                      lse_rows<false, T, NW * 64>(p, x, sQ, sRun, r, n, r == r0);
    };
    for (int r = r0; r < n;) {
#pragma unroll
        for (int x = 0; x < S; ++x) {
            if (r >= n) break;
            rows(k[x], r);
            if (r + S * step < n) load_k_rows<T>(k[x], kb, r + S * step, n16, n);
            r += step;
        }
    }
    // fold the four row groups of the wavefront, then the wavefronts (through the LDS of the queries)
    __syncthreads();
    float* sM = reinterpret_cast<float*>(window_lds);                // [NW][ncol]
    float* sL = sM + NW * ncol;
    static_assert(2 * NW * sizeof(float) <= kQStride * sizeof(uint16_t), "the wavefronts' pairs fit where the queries were");
    for (int cb = 0; cb < ncb; ++cb) {
        const float2 run = r0 < n ? sRun[cb * NW * 64 + tid] : make_float2(-INFINITY, 0.f);
        const float M = max_xor32(max_xor16(run.x));
        const float a = run.x == -INFINITY ? 0.f : fast_exp2(run.x - M);
        const float L = sum_xor32(sum_xor16(run.y * a));
        if (c4 == 0) { sM[w * ncol + cb * 16 + n16] = M; sL[w * ncol + cb * 16 + n16] = L; }
    }
    __syncthreads();
    const int64_t bg = (int64_t)b * p.Hkv + g;
    float* part = p.part + ((bg * p.nch + c) * ncol) * 2;
    for (int col = tid; col < ncol; col += NW * 64) {
        float M = sM[col], L = sL[col];
#pragma unroll
        for (int ww = 1; ww < NW; ++ww) merge_ml(M, L, sM[ww * ncol + col], sL[ww * ncol + col]);
        *reinterpret_cast<float2*>(part + col * 2) = make_float2(M, L);
    }
}

// What a column's scores are normalised with: vote = 2^(s - maximum) / sum.  With lse = maximum + ln sum as two floats and
// e^(s - lse) an exponent took two subtractions and two products instead of one multiply-add.  Largest relative error of votes of
// at least 1e-3 of the largest, whole-number products (exact), for e^(s - lse) / for maxima and sums of scores rounded in pass 1 alone / now:
// scores to 100: 7e-7 and less / 2.2e-6 / 9e-7, to 400: 2.7e-6 / 4.2e-6 / 8e-7, to 1000: 1.1e-5 / 1.7e-5 / 8e-7; normal keys (scores of a
// few units, 32768 rows, 32 queries, 2-norm): 1.7e-7 / 8.0e-8 / 8.0e-8.  Whole call, us, the first / the last: 32768 rows, 32 queries 61.2 / 60.2,
// 28 heads over 4, 30000 rows 73.1 / 70.7, 64 over 8, 20000 rows 87.5 / 84.6, 8 sequences of 2000 rows 48.1 / 46.5.
__device__ __forceinline__ float2 column_norm(const WindowParams& p, int col, int n, float M, double L) {
    // (a column that does not exist was summed like the others; one without a finite score has no sum)
    return (M != -INFINITY && column_limit(p, col, n) >= 0) ? make_float2(M, (float)(1.0 / L)) : make_float2(0.f, 0.f);
}

// Maximum and 1 / sum of every column from the per-workgroup pairs: one workgroup per (block of 16 columns,
// sequence, KV head); thread (n16, cl) folds the pairs of column n16 from workgroups cl, cl + 16,
// ...; thread (n16, 0) folds the 16 results, the sum in fp64.
__global__ __launch_bounds__(256)
void window_lse_merge_kernel(const WindowParams p) {
    const int cb = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    if (p.pred != nullptr && p.pred[b] != p.pred_val) return;
    const int n = min(max(min(p.seq_lens[b], p.cap), 0), p.max_rows);
    if (n == 0) return;
    const int nchunks = window_workgroups(p, n);
    const int ncol = p.ncb * 16;
    const int n16 = threadIdx.x & 15, cl = threadIdx.x >> 4;
    const int col = cb * 16 + n16;
    const int64_t bg = (int64_t)b * p.Hkv + g;
    const float* part = p.part + (bg * p.nch * ncol + col) * 2;
    float m = -INFINITY, l = 0.f;
    for (int c0 = cl; c0 < nchunks; c0 += 64) {            // four loads in flight
        float2 ml[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int c = c0 + 16 * u;
            ml[u] = c < nchunks ? *reinterpret_cast<const float2*>(part + (int64_t)c * ncol * 2) : make_float2(-INFINITY, 0.f);
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) merge_ml(m, l, ml[u].x, ml[u].y);
    }
    __shared__ float sM[16][16], sL[16][16];
    sM[cl][n16] = m; sL[cl][n16] = l;
    __syncthreads();
    if (cl == 0) {
        float M = -INFINITY;
#pragma unroll
        for (int x = 0; x < 16; ++x) M = fmaxf(M, sM[x][n16]);
        double L = 0.0;
#pragma unroll
        for (int x = 0; x < 16; ++x)
            if (sM[x][n16] != -INFINITY) L += (double)fast_exp2(sM[x][n16] - M) * (double)sL[x][n16];
        *reinterpret_cast<float2*>(p.lse + (bg * ncol + col) * 2) = column_norm(p, col, n, M, L);
    }
}

// Sum over the lanes of a row of 16 that hold the same head (lane % gp), on the DPP operand path.
__device__ __forceinline__ float sum_queries(float v, int gp) {
    if (gp <= 8) v += dpp_move_f<kDppRor8>(v);
    if (gp <= 4) v += dpp_move_f<kDppRor4>(v);
    if (gp <= 2) v += dpp_move_f<kDppXor2>(v);
    if (gp <= 1) v += dpp_move_f<kDppXor1>(v);
    return v;
}

// Pass 2.
template <bool MASKED, int T>
__device__ __forceinline__ void vote_rows(const WindowParams& p, const u32x4 (&k)[T][4], const uint16_t* sQ,
                                          const float2* sLse, float* vrow, int r, int n) {
    const int lane = threadIdx.x & 63, n16 = lane & 15, c4 = lane >> 4;
    float v[T][4];
#pragma unroll
    for (int e = 0; e < 4 * T; ++e) v[e >> 2][e & 3] = 0.f;
    auto block = [&](auto masked, int cb) {
        constexpr bool kMasked = decltype(masked)::value;
        float x[T][4];
        block_products<kMasked, T>(k, sQ, cb, n16, c4, r, kMasked ? column_limit(p, cb * 16 + n16, n) : 0, x);
        const float2 norm = sLse[cb * 16 + n16];
#pragma unroll
        for (int e = 0; e < 4 * T; ++e)            // (masked: 2^-inf = 0; no such column: times 0)
            v[e >> 2][e & 3] = fmaf(fast_exp2(fmaf(x[e >> 2][e & 3], p.scale2, -norm.x)), norm.y, v[e >> 2][e & 3]);
    };
    // A last block that the queries do not fill has columns which are added to real ones below; their zero queries' scores
    // are NaN where a key is infinite, so that block is masked also where every query sees every row.
    const int full = MASKED ? p.ncb : (p.W << p.gp_shift) >> 4;
#pragma unroll 1
    for (int cb = 0; cb < full; ++cb) block(std::integral_constant<bool, MASKED>{}, cb);
    if (!MASKED && full < p.ncb) block(std::true_type{}, full);
    // lanes n16, n16 + Gp, n16 + 2 Gp ... hold the same head for different queries
    const int gp = 1 << p.gp_shift;
#pragma unroll
    for (int e = 0; e < 4 * T; ++e) v[e >> 2][e & 3] = sum_queries(v[e >> 2][e & 3], gp);
    if (n16 < p.G) {
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const int first = r + t * 16 + 4 * c4;
            if (p.v_vec && first + 4 <= n) {
                *reinterpret_cast<float4*>(vrow + first) = make_float4(v[t][0], v[t][1], v[t][2], v[t][3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (first + i < n) vrow[first + i] = v[t][i];
            }
        }
    }
}

// FOLD: the (max, sum) pairs of pass 1 are folded here, up to kFoldHeld per thread, while the rows are on their way; where there
// are more (or the columns are no power of two) by window_lse_merge_kernel, a launch of 4.6 us between the passes.  Whole
// call with that launch / folded here, us, 32 heads over 8: 1100 rows, 32 queries 28.6 / 26.8; 3000 rows 33.2 / 31.2; 8 sequences of
// 2000 rows 46.5 / 44.7; 32768 rows, 8 queries 49.8 / 48.6, 32 queries 60.2 / 59.5 (every workgroup reads 64 KB of pairs there).
constexpr int kFoldHeld = 16;
template <int T, int S, int NW, bool FOLD>
__global__ __launch_bounds__(NW * 64, 4)
void window_vote_kernel(const WindowParams p) {
    const int ncol = p.ncb * 16;
    const int c = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
    if (p.pred != nullptr && p.pred[b] != p.pred_val) return;
    const int n = min(max(min(p.seq_lens[b], p.cap), 0), p.max_rows);
    if (n == 0 || c >= window_workgroups(p, n)) return;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int n16 = lane & 15, c4 = lane >> 4;
    uint16_t* sQ = reinterpret_cast<uint16_t*>(window_lds);
    float2* sLse = reinterpret_cast<float2*>(window_lds + (size_t)ncol * kQStride * 2);   // [ncol]
    const int64_t bg = (int64_t)b * p.Hkv + g;

    const uint16_t* kb = p.k + (int64_t)b * p.s_b + (int64_t)g * p.s_h + c4 * 8;
    const int step = p.nch * NW * 16 * T, r0 = (c * NW + w) * 16 * T;
    uint4 held[kQHeld];
    u32x4 k[S][T][4];
    const float2* lse_of = reinterpret_cast<const float2*>(p.lse) + bg * ncol;
    const float2 my_lse = !FOLD && tid < ncol ? lse_of[tid] : make_float2(0.f, 0.f);
    static_assert(NW * 64 >= 32 * RK_MAX_GROUP, "a thread per column");
    request_queries<NW * 64>(p, b, g, n, held);
    // column tid mod ncol (ncol is a power of two where FOLD is used), every groups-th workgroup's pair from tid / ncol on
    const int fold_col = tid & (ncol - 1), fold_lg = 31 - __builtin_clz(ncol), groups = NW * 64 >> fold_lg, fold_g = tid >> fold_lg;
    const int nchunks = window_workgroups(p, n);
    float2 pairs[kFoldHeld];
    if constexpr (FOLD) {
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(p.part + bg * p.nch * ncol * 2, 0, nchunks * ncol * 8, 0x00020000);
#pragma unroll
        for (int u = 0; u < kFoldHeld; ++u)       // (behind the last workgroup's: zeros, a sum of nothing)
            pairs[u] = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(rp, ((fold_g + u * groups) * ncol + fold_col) * 8, 0, 0));
    }
#pragma unroll
    for (int x = 0; x < S; ++x)
        if (r0 + x * step < n) load_k_rows<T>(k[x], kb, r0 + x * step, n16, n);
    store_queries<NW * 64>(p, b, g, n, ncol, held, sQ);
    if constexpr (FOLD) {
        float2* sMl = sLse + ncol;                // [NW * 64]
        double* sSum = reinterpret_cast<double*>(sMl);
        float M = -INFINITY;
#pragma unroll
        for (int u = 0; u < kFoldHeld; ++u) M = fmaxf(M, pairs[u].y != 0.f ? pairs[u].x : -INFINITY);
        double L = 0.0;
#pragma unroll
        for (int u = 0; u < kFoldHeld; ++u)
            if (pairs[u].y != 0.f && pairs[u].x != -INFINITY) L += (double)fast_exp2(pairs[u].x - M) * (double)pairs[u].y;
        float* sM = reinterpret_cast<float*>(sSum + NW * 64);
        sSum[tid] = L; sM[tid] = M;
        lds_barrier();
        if (tid < ncol) {
            float all = -INFINITY;
            for (int x = 0; x < groups; ++x) all = fmaxf(all, sM[x * ncol + tid]);
            double sum = 0.0;
            for (int x = 0; x < groups; ++x)
                if (sM[x * ncol + tid] != -INFINITY) sum += (double)fast_exp2(sM[x * ncol + tid] - all) * sSum[x * ncol + tid];
            sLse[tid] = column_norm(p, tid, n, all, sum);
        }
        lds_barrier();
    } else {
        if (tid < ncol) sLse[tid] = my_lse;
        __syncthreads();
    }
    float* vrow = p.votes + ((int64_t)b * p.Hq + (int64_t)g * p.G + (n16 < p.G ? n16 : 0)) * p.v_stride;
    auto rows = [&](const u32x4 (&x)[T][4], int r) {
        if (r + 16 * T > n - p.W) vote_rows<true, T>(p, x, sQ, sLse, vrow, r, n);
        else                      vote_rows<false, T>(p, x, sQ, sLse, vrow, r, n);
    };
    for (int r = r0; r < n;) {
#pragma unroll
        for (int x = 0; x < S; ++x) {
            if (r >= n) break;
            rows(k[x], r);
            if (r + S * step < n) load_k_rows<T>(k[x], kb, r + S * step, n16, n);
            r += step;
        }
    }
}

template <int T, int S, int NW>
static int launch_window(const WindowParams& p, int batch, hipStream_t st) {
    const size_t ncol = (size_t)p.ncb * 16;
    const size_t lds1 = ncol * kQStride * 2 + (size_t)p.ncb * NW * 64 * sizeof(float2);
    const bool fold = (ncol & (ncol - 1)) == 0 && ncol <= (size_t)NW * 64 && (size_t)p.nch * ncol <= (size_t)kFoldHeld * NW * 64;
    const size_t lds2 = ncol * kQStride * 2 + ncol * sizeof(float2) + (fold ? NW * 64 * (sizeof(double) + sizeof(float)) : 0);
    const size_t lds = lds1 > lds2 ? lds1 : lds2;
    static size_t lds_allowed = 48 * 1024;       // grows monotonically
    if (lds > lds_allowed) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&window_lse_kernel<T, S, NW>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&window_vote_kernel<T, S, NW, true>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&window_vote_kernel<T, S, NW, false>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
            (void)hipGetLastError();
            return RK_ERR_UNSUPPORTED;
        }
        lds_allowed = lds;
    }
    dim3 grid(p.nch, p.Hkv, batch);
    hipLaunchKernelGGL((window_lse_kernel<T, S, NW>), grid, dim3(NW * 64), lds1, st, p);
    int rc = launch_status();
    if (rc != RK_OK) return rc;
    if (fold) {
        hipLaunchKernelGGL((window_vote_kernel<T, S, NW, true>), grid, dim3(NW * 64), lds2, st, p);
        return launch_status();
    }
    hipLaunchKernelGGL(window_lse_merge_kernel, dim3(p.ncb, p.Hkv, batch), dim3(256), 0, st, p);
    if ((rc = launch_status()) != RK_OK) return rc;
    hipLaunchKernelGGL((window_vote_kernel<T, S, NW, false>), grid, dim3(NW * 64), lds2, st, p);
    return launch_status();
}

}  // namespace rk

using namespace rk;

extern "C" int rk_window_select(const rk_geom* geom, const void* q_win, int32_t window, rk_kv full,
                                const int32_t* seq_lens, int32_t max_len,
                                float* votes, int64_t v_stride,
                                int32_t k, int32_t pool_w, int32_t agg,
                                int32_t* idx, float* sel_scores,
                                const int32_t* pred, int32_t pred_val,
                                void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!q_win || !seq_lens || !idx || max_len <= 0 || k <= 0 || window <= 0) return RK_ERR_INVALID_ARG;
    if (window > RK_MAX_WINDOW) return RK_ERR_UNSUPPORTED;
    if (!aligned16(q_win)) return RK_ERR_INVALID_ARG;
    if ((rc = check_kv(full, false)) != RK_OK) return rc;
    if (votes && (v_stride < max_len || ((uintptr_t)votes & 3u))) return RK_ERR_INVALID_ARG;
    if ((rc = check_select_args(k, pool_w, agg, max_len)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, k, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    hipStream_t st = (hipStream_t)stream;

    const int G = geom->n_q_heads / geom->n_kv_heads;
    int gp_shift = 0;
    while ((1 << gp_shift) < G) ++gp_shift;
    const int blocks = ((window << gp_shift) + 15) / 16;           // blocks of 16 columns in use
    const int ncb = blocks;
    // the per-workgroup (max, sum) pairs borrow the partial-output area, the column lse the area of
    // the decode kernels' (max, sum) pairs: both are free between calls
    if ((size_t)ncb * 16 * 2 > (size_t)G * kD || (size_t)ncb * 16 > (size_t)kMaxChunks * G) return RK_ERR_UNSUPPORTED;

    WindowParams p{};
    p.q = (const uint16_t*)q_win;
    p.k = (const uint16_t*)full.k; p.s_b = full.stride_b; p.s_h = full.stride_h; p.cap = (int32_t)full.capacity;
    p.seq_lens = seq_lens; p.max_rows = max_len;
    p.W = window; p.G = G; p.gp_shift = gp_shift;
    const WindowForm form = window_form(max_len, (int64_t)geom->batch * geom->n_kv_heads, ncb, ws.max_chunks);
    p.wg_rows = form.wg_rows; p.nch = form.nch;
    p.Hq = geom->n_q_heads; p.Hkv = geom->n_kv_heads;
    p.scale2 = (float)(fabs((double)geom->scale) * 1.4426950408889634);
    if (p.scale2 == 0.f) p.scale2 = FLT_MIN;                       // (a masked row's -inf times 0 would be NaN; 2^(x FLT_MIN) is 1)
    p.q_sign = geom->scale < 0.f ? 0x80008000u : 0u;
    p.part = ws.part_o; p.lse = ws.part_ml;
    if (votes) { p.votes = votes; p.v_stride = v_stride; }
    else       { p.votes = ws.scores; p.v_stride = pooled_row_stride(max_len); }
    p.v_vec = ((p.v_stride % 4 == 0) && aligned16(p.votes)) ? 1 : 0;
    p.pred = pred; p.pred_val = pred_val;
    p.ncb = ncb;
    rc = form.T == 1 ? launch_window<1, 1, 8>(p, geom->batch, st)
       : form.T == 2 ? launch_window<2, 2, 4>(p, geom->batch, st) : launch_window<4, 1, 8>(p, geom->batch, st);
    if (rc != RK_OK) return rc;
    if ((rc = pool_stage(geom, p.votes, p.v_stride, seq_lens, max_len, pool_w, agg, pred, pred_val, ws, st)) != RK_OK) return rc;
    return select_stage(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, st);
}
