// The H2O comparison policy on the library's attention step: rk_h2o_append, rk_h2o_update,
// rk_h2o_step (Section 3 "Comparison systems"; Appendix A.1 "Baseline Settings").
//
// A step = append the new token's rows to the policy's cache, attend over the whole cache with
// the scores returned (at most budget + 1 rows), then one small kernel per (sequence, KV head): add the
// group-aggregated scores to the running totals and, when the cache is over its budget, drop the token
// with the lowest total among those that are not recent.  Slots are not kept in token order (attention does not
// care): the newest token, always in the last slot, moves into the slot of the dropped one, so the
// cache stays dense without shifting rows.  rk_h2o_step takes two launches: the attention reads the new row from
// the caller's tensors, and the kernel that follows merges the output, updates the totals and stores the row.
// The parts as calls of their own (and new rows that are not 16-byte aligned) go append, rk_full_attn's kernels, update;
// rows are shared out and partial results summed in the same order either way, so the results have the same bits.
#include "rk_internal.h"
#include "rk_device.h"

namespace rk {

constexpr int kH2oThreads = 1024;

__global__ __launch_bounds__(64)
void h2o_append_kernel(rk_h2o_state st, const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new,
                       const int32_t* __restrict__ seq_lens, int32_t Hkv, int64_t meta_stride) {
    const int g = blockIdx.x, b = blockIdx.y, lane = threadIdx.x;
    const int cap = (int)st.cache.capacity;
    const int slot = min(max(st.n_rows[b], 0), cap - 1);
    const int64_t bg = (int64_t)b * Hkv + g;
    const uint32_t* ks = reinterpret_cast<const uint32_t*>(k_new + bg * kD);
    const uint32_t* vs = reinterpret_cast<const uint32_t*>(v_new + bg * kD);
    uint16_t* kc = (uint16_t*)st.cache.k + (int64_t)b * st.cache.stride_b + (int64_t)g * st.cache.stride_h + (int64_t)slot * kD;
    uint16_t* vc = (uint16_t*)st.cache.v + (int64_t)b * st.cache.stride_b + (int64_t)g * st.cache.stride_h + (int64_t)slot * kD;
    reinterpret_cast<uint32_t*>(kc)[lane] = ks[lane];
    reinterpret_cast<uint32_t*>(vc)[lane] = vs[lane];
    if (lane == 0) {
        st.total[bg * meta_stride + slot] = 0.f;
        st.pos[bg * meta_stride + slot] = seq_lens[b] - 1;
        st.n_attend[b] = slot + 1;                 // every head of the sequence writes the same value
    }
}

// 64-bit minimum over the workgroup; `red` holds kH2oThreads / 64 words.  Every thread gets it.
__device__ __forceinline__ uint64_t block_min_u64(uint64_t v, uint64_t* red) {
#pragma unroll
    for (int m = 1; m < 64; m <<= 1) {
        const uint64_t o = __shfl_xor(v, m);
        v = o < v ? o : v;
    }
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    uint64_t r = red[0];
    for (int i = 1; i < kH2oThreads / 64; ++i) r = red[i] < r ? red[i] : r;
    return r;
}

__global__ __launch_bounds__(kH2oThreads)
void h2o_update_kernel(rk_h2o_state st, const float* __restrict__ weights, int64_t w_stride, int32_t max_rows,
                       int32_t Hq, int32_t Hkv, int32_t G, int32_t budget, int32_t recent, int32_t agg,
                       int32_t* __restrict__ dropped, int64_t meta_stride) {
    const int g = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int cap = (int)st.cache.capacity;
    const int n = min(min(max(st.n_attend[b], 0), cap), max_rows);
    const int64_t bg = (int64_t)b * Hkv + g;
    float* total = st.total + bg * meta_stride;
    int32_t* pos = st.pos + bg * meta_stride;
    const float* wg = weights + ((int64_t)b * Hq + (int64_t)g * G) * w_stride;
    __shared__ uint64_t red[kH2oThreads / 64];
    __shared__ int sVictim;
    const bool over = n > budget;
    const int newest = n > 0 ? pos[n - 1] : 0;
    uint64_t best = ~0ull;
    for (int j = tid; j < n; j += kH2oThreads) {
        float a = -INFINITY;
        for (int gi = 0; gi < G; ++gi) a = aggregate(a, wg[(int64_t)gi * w_stride + j], gi, agg);
        if (agg == RK_AGG_MEAN) a = __fdiv_rn(a, (float)G);
        const float t = __fadd_rn(total[j], a);
        total[j] = t;
        const int pj = pos[j];
        if (over && pj <= newest - recent) {       // lowest total first, the older token on equal totals
            const uint64_t key = ((uint64_t)key_of(t) << 32) | (uint32_t)pj;
            best = key < best ? key : best;
        }
    }
    if (tid == 0) sVictim = -1;
    best = block_min_u64(best, red);               // has a barrier after the write of sVictim
    int32_t gone = -1;
    if (over && best != ~0ull) {
        gone = (int32_t)(uint32_t)best;
        for (int j = tid; j < n; j += kH2oThreads)
            if (pos[j] == gone) sVictim = j;       // positions are unique within a cache
        __syncthreads();
        const int v = sVictim, last = n - 1;
        if (v >= 0 && v != last) {
            uint16_t* kc = (uint16_t*)st.cache.k + (int64_t)b * st.cache.stride_b + (int64_t)g * st.cache.stride_h;
            uint16_t* vc = (uint16_t*)st.cache.v + (int64_t)b * st.cache.stride_b + (int64_t)g * st.cache.stride_h;
            if (tid < 64)        reinterpret_cast<uint32_t*>(kc + (int64_t)v * kD)[tid] = reinterpret_cast<const uint32_t*>(kc + (int64_t)last * kD)[tid];
            else if (tid < 128)  reinterpret_cast<uint32_t*>(vc + (int64_t)v * kD)[tid - 64] = reinterpret_cast<const uint32_t*>(vc + (int64_t)last * kD)[tid - 64];
            else if (tid == 128) { total[v] = total[last]; pos[v] = pos[last]; }
        }
    }
    if (tid == 0) {
        if (dropped) dropped[bg] = gone;
        st.n_rows[b] = gone >= 0 ? n - 1 : n;      // every head of the sequence writes the same value
    }
}

// What follows the attention of a step in one launch, one workgroup per (sequence, KV head): the log-sum-exp of the
// group's heads from the partial results, the output merge, the weights from the raw scores (one exponential per
// row where the group takes its maximum), the totals, the drop rule, and the new token's rows into the cache.
// A chain of dependent steps on one CU: what it costs is round trips and barriers, so everything it reads is
// requested before the first wait and the output merge runs between the requests and the weights.
// Measured, 32 heads over 8, 2048 rows, us per launch: 4 sequences: append 2.9 + attention 12.6 + merge and weights 5.9 +
// update 8.0 -> attention (the new row read where the caller has it) 8.8 + this 7.0; one sequence 5.7 + 7.0.  (A workgroup
// of its own for the new row, and the small cache in wavefronts of one tile: 10.3, and other bits than the parts.)
constexpr int kH2oHeld = 4;                        // rows per thread requested up front: 4096 in all
template <int G>
__global__ __launch_bounds__(kH2oThreads)
void h2o_finish_kernel(rk_h2o_state st, const float* __restrict__ scores, int64_t s_stride, const float* __restrict__ part_ml,
                       const float* __restrict__ part_o, int32_t max_chunks, int32_t nch, const int32_t* __restrict__ counters, int32_t max_rows,
                       const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new, const int32_t* __restrict__ seq_lens,
                       int32_t Hkv, int32_t budget, int32_t recent, int32_t agg, uint16_t* __restrict__ out,
                       int32_t* __restrict__ dropped, int64_t meta_stride) {
    const int g = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int cap = (int)st.cache.capacity;
    const int attend = min(max(st.n_attend[b], 1), cap), slot = attend - 1;      // the new token's slot
    const int n = min(attend, max_rows);
    const int64_t bg = (int64_t)b * Hkv + g;
    float* total = st.total + bg * meta_stride;
    int32_t* pos = st.pos + bg * meta_stride;
    const float* sg = scores + bg * G * s_stride;
    // (counters: a ragged batch, whose shares the attention left there; NULL: all sequences share rows out alike)
    const int nchunks = counters != nullptr ? stored_chunks(counters, bg) : max(1, min(nch, (n + kMinChunk - 1) / kMinChunk));

    __shared__ uint64_t red[kH2oThreads / 64];
    __shared__ int sVictim;
    __shared__ __attribute__((aligned(8))) float sLse[G][2];
    __shared__ float sW[G][kMaxChunks];
    __shared__ float sInv[G];
    // four sums over every fourth partial result each, as in the merge of rk_full_attn, so that the output has its bits
    constexpr int kPairs = G * kD / 2, kSums = 4;                                // threads of a set: two dims of a head each
    constexpr int kSets = kSums * kPairs <= kH2oThreads ? kSums : kSums / 2;     // sets of threads, kSums / kSets sums each
    static_assert(kSets * kPairs <= kH2oThreads, "sets of partial results");
    __shared__ __attribute__((aligned(8))) float2 sAcc[kSums][kPairs];

    // ---- requests: the chunk statistics, the first scores, totals and positions, the first partial outputs ----
    constexpr int kStat = kMaxChunks / 64;
    float m[kStat], l[kStat];
    if (w < G) {
#pragma unroll
        for (int u = 0; u < kStat; ++u) {
            m[u] = -INFINITY; l[u] = 0.f;
            const int c = lane + 64 * u;
            if (c < nchunks) {
                const float2 t2 = *reinterpret_cast<const float2*>(part_ml + ((bg * kMaxChunks + c) * G + w) * 2);
                m[u] = t2.x; l[u] = t2.y;
            }
        }
    }
    float sc[kH2oHeld][G], tot[kH2oHeld];
    int ps[kH2oHeld];
    auto request = [&](int u, int j) {
        const bool in = j < n;
        if constexpr (G == 4) {                      // the four heads of a row side by side
            const float4 v4 = in ? *reinterpret_cast<const float4*>(sg + (int64_t)j * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
            sc[u][0] = v4.x; sc[u][1] = v4.y; sc[u][2] = v4.z; sc[u][3] = v4.w;
        } else {
#pragma unroll
            for (int gi = 0; gi < G; ++gi) sc[u][gi] = in ? sg[(int64_t)gi * s_stride + j] : 0.f;
        }
        tot[u] = in && j != slot ? total[j] : 0.f;
        ps[u] = in && j != slot ? pos[j] : 0;
    };
#pragma unroll
    for (int u = 0; u < kH2oHeld; ++u) request(u, u * kH2oThreads + tid);
    const int new_pos = seq_lens[b] - 1;
    const int newest = n - 1 == slot ? new_pos : pos[n - 1];
    const int set = tid / kPairs, e2 = tid - set * kPairs, gi_out = 2 * e2 / kD;
    const float* po = part_o + bg * max_chunks * G * kD + 2 * e2;
    constexpr int kOut = 8;                          // partial outputs per round trip and thread
    float2 o[kOut];
    auto request_out = [&](int c0) {
#pragma unroll
        for (int u = 0; u < kOut; ++u)
            o[u] = *reinterpret_cast<const float2*>(po + (int64_t)min(c0 + u * kSums, nchunks - 1) * G * kD);
    };
    if (set < kSets) request_out(set);
    // the new row, two dims per lane: wavefront 14 its key, wavefront 15 its value
    uint32_t fresh = 0;
    if (w >= 14) fresh = reinterpret_cast<const uint32_t*>((w == 14 ? k_new : v_new) + bg * kD)[lane];

    // ---- lse of the heads, fp64, one wavefront each ----
    if (w < G) {
        float M = m[0];
#pragma unroll
        for (int u = 1; u < kStat; ++u) M = fmaxf(M, m[u]);
        M = wave_max(M);
        double L = 0.0;
#pragma unroll
        for (int u = 0; u < kStat; ++u) {
            if (64 * u >= nchunks) break;
            const float wgt = m[u] == -INFINITY ? 0.f : fast_exp2((m[u] - M) * kLog2e);
            if (lane + 64 * u < nchunks) sW[w][lane + 64 * u] = wgt;
            L += wave_sum((double)wgt * (double)l[u]);
        }
        if (lane == 0) {
            float hi = -INFINITY, lo = 0.f;
            if (L > 0.0) {
                const double l64 = (double)M + log(L);
                hi = (float)l64;
                lo = (float)(l64 - (double)hi);
            }
            sLse[w][0] = hi; sLse[w][1] = lo;
            sInv[w] = L > 0.0 ? (float)L : 0.f;
        }
    }
    if (tid == 0) sVictim = -1;
    __syncthreads();

    // ---- output: sum x takes the partial results x, x + 4, x + 8 ... ----
    if (set < kSets) {
#pragma unroll
        for (int x = set; x < kSums; x += kSets) {
            float2 acc = make_float2(0.f, 0.f);
            for (int c0 = x; c0 < nchunks; c0 += kOut * kSums) {
                if (c0 != set) request_out(c0);
#pragma unroll
                for (int u = 0; u < kOut; ++u) {
                    const int c = c0 + u * kSums;
                    const float wc = c < nchunks ? sW[gi_out][c] : 0.f;
                    acc.x = fmaf(wc, o[u].x, acc.x);
                    acc.y = fmaf(wc, o[u].y, acc.y);
                }
            }
            sAcc[x][e2] = acc;
        }
    }

    // ---- totals, and the lowest of the old ones ----
    const bool over = n > budget;
    uint64_t best = ~0ull;
    float tol = 1.5e-5f;
#pragma unroll
    for (int gi = 0; gi < G; ++gi) tol += fabsf(sLse[gi][1]);
    auto row = [&](int u, int j) {
        float a;
        if (agg == RK_AGG_MAX) {
            a = max_weight<G>(sc[u], sLse, tol);
        } else {
            a = -INFINITY;
#pragma unroll
            for (int gi = 0; gi < G; ++gi) a = aggregate(a, weight_of(sc[u][gi], -sLse[gi][0], sLse[gi][1]), gi, agg);
            if (agg == RK_AGG_MEAN) a = __fdiv_rn(a, (float)G);
        }
        if (j >= n) return;
        const float t = __fadd_rn(tot[u], a);
        total[j] = t;
        const int pj = j == slot ? new_pos : ps[u];
        if (j == slot) pos[j] = new_pos;
        if (over && pj <= newest - recent) {       // lowest total first, the older token on equal totals
            const uint64_t key = ((uint64_t)key_of(t) << 32) | (uint32_t)pj;
            best = key < best ? key : best;
        }
    };
    for (int j0 = 0; j0 < n; j0 += kH2oHeld * kH2oThreads) {
        if (j0 != 0) {
#pragma unroll
            for (int u = 0; u < kH2oHeld; ++u) request(u, j0 + u * kH2oThreads + tid);
        }
#pragma unroll
        for (int u = 0; u < kH2oHeld; ++u)
            if (j0 + u * kH2oThreads < n) row(u, j0 + u * kH2oThreads + tid);
    }
    best = block_min_u64(best, red);               // (a barrier: the sums of the sets are in LDS as well)
    if (tid < kPairs) {
        float2 acc = sAcc[0][tid];
#pragma unroll
        for (int x = 1; x < kSums; ++x) { acc.x += sAcc[x][tid].x; acc.y += sAcc[x][tid].y; }
        const float L = sInv[2 * tid / kD];
        const float ox = L > 0.f ? acc.x / L : 0.f, oy = L > 0.f ? acc.y / L : 0.f;
        const uint32_t pair = (uint32_t)f32_to_bf16(ox) | ((uint32_t)f32_to_bf16(oy) << 16);
        uint16_t* dst = out + bg * G * kD + 2 * tid;                    // 2-byte alignment is all that is asked of out
        dst[0] = (uint16_t)pair; dst[1] = (uint16_t)(pair >> 16);
    }
    int32_t gone = -1;
    int v = -1;
    if (over && best != ~0ull) {
        gone = (int32_t)(uint32_t)best;
        for (int j = tid; j < n; j += kH2oThreads)
            if ((j == slot ? new_pos : pos[j]) == gone) sVictim = j;     // positions are unique within a cache
        __syncthreads();
        v = sVictim;
    }
    // the new token's rows to its slot; the last row (the new one, unless the cache was over its budget) also to
    // the dropped one's
    const int last = n - 1;
    const bool move = v >= 0 && v != last;
    if (w >= 14) {
        uint16_t* rows = (uint16_t*)(w == 14 ? st.cache.k : st.cache.v) + (int64_t)b * st.cache.stride_b + (int64_t)g * st.cache.stride_h;
        reinterpret_cast<uint32_t*>(rows + (int64_t)slot * kD)[lane] = fresh;
        if (move) {
            const uint32_t x = last == slot ? fresh : reinterpret_cast<const uint32_t*>(rows + (int64_t)last * kD)[lane];
            reinterpret_cast<uint32_t*>(rows + (int64_t)v * kD)[lane] = x;
        }
    } else if (tid == 0) {
        if (slot >= n) { total[slot] = 0.f; pos[slot] = new_pos; }      // appended, but beyond what the step attends over
        if (move) { total[v] = total[last]; pos[v] = last == slot ? new_pos : pos[last]; }
        if (dropped) dropped[bg] = gone;
        st.n_rows[b] = gone >= 0 ? n - 1 : n;      // every head of the sequence writes the same value
    }
}

static int check_h2o(const rk_geom* geom, const rk_h2o_state& st, int32_t budget, int32_t recent) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if ((rc = check_kv(st.cache)) != RK_OK) return rc;
    if (!st.total || !st.pos || !st.n_rows || !st.n_attend) return RK_ERR_INVALID_ARG;
    if (budget <= 0 || recent < 0 || recent >= budget) return RK_ERR_INVALID_ARG;
    if (st.cache.capacity < (int64_t)budget + 1) return RK_ERR_INVALID_ARG;
    return RK_OK;
}

static int append_stage(const rk_geom* geom, const rk_h2o_state& st, const void* k_new, const void* v_new,
                        const int32_t* seq_lens, hipStream_t s) {
    hipLaunchKernelGGL(h2o_append_kernel, dim3(geom->n_kv_heads, geom->batch), dim3(64), 0, s, st,
                       (const uint16_t*)k_new, (const uint16_t*)v_new, seq_lens, geom->n_kv_heads, st.cache.capacity);
    return launch_status();
}

static int update_stage(const rk_geom* geom, const rk_h2o_state& st, const float* weights, int64_t w_stride,
                        int32_t max_rows, int32_t budget, int32_t recent, int32_t agg, int32_t* dropped, hipStream_t s) {
    hipLaunchKernelGGL(h2o_update_kernel, dim3(geom->n_kv_heads, geom->batch), dim3(kH2oThreads), 0, s, st,
                       weights, w_stride, max_rows, geom->n_q_heads, geom->n_kv_heads, geom->n_q_heads / geom->n_kv_heads,
                       budget, recent, agg, dropped, st.cache.capacity);
    return launch_status();
}

}  // namespace rk

using namespace rk;

extern "C" int rk_h2o_append(const rk_geom* geom, rk_h2o_state state, const void* k_new, const void* v_new,
                             const int32_t* seq_lens, int32_t budget, void* stream) {
    int rc = check_h2o(geom, state, budget, 0);
    if (rc != RK_OK) return rc;
    if (!k_new || !v_new || !seq_lens || ((uintptr_t)k_new & 3u) || ((uintptr_t)v_new & 3u)) return RK_ERR_INVALID_ARG;
    return append_stage(geom, state, k_new, v_new, seq_lens, (hipStream_t)stream);
}

extern "C" int rk_h2o_update(const rk_geom* geom, rk_h2o_state state, const float* weights, int64_t w_stride,
                             int32_t budget, int32_t recent, int32_t agg, int32_t* dropped, void* stream) {
    int rc = check_h2o(geom, state, budget, recent);
    if (rc != RK_OK) return rc;
    if (!weights || w_stride < (int64_t)budget + 1 || ((uintptr_t)weights & 3u)) return RK_ERR_INVALID_ARG;
    if (agg < RK_AGG_MAX || agg > RK_AGG_FIRST) return RK_ERR_UNSUPPORTED;
    return update_stage(geom, state, weights, w_stride, budget + 1, budget, recent, agg, dropped, (hipStream_t)stream);
}

extern "C" int rk_h2o_step(const rk_geom* geom, rk_h2o_state state, const void* q,
                           const void* k_new, const void* v_new, const int32_t* seq_lens,
                           int32_t budget, int32_t recent, int32_t agg,
                           void* out, int32_t* dropped,
                           void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_h2o(geom, state, budget, recent);
    if (rc != RK_OK) return rc;
    if (!q || !out || !k_new || !v_new || !seq_lens) return RK_ERR_INVALID_ARG;
    if (!aligned16(q) || ((uintptr_t)out & 1u) || ((uintptr_t)k_new & 3u) || ((uintptr_t)v_new & 3u)) return RK_ERR_INVALID_ARG;
    if (agg < RK_AGG_MAX || agg > RK_AGG_FIRST) return RK_ERR_UNSUPPORTED;
    const int32_t max_rows = budget + 1;
    Workspace ws;
    if ((rc = check_workspace(geom, max_rows, 0, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int nch = h2o_split_workgroups(geom, max_rows);
    if (!aligned16(k_new) || !aligned16(v_new)) {      // the attention reads the new row where it is, in 16-byte loads
        if ((rc = append_stage(geom, state, k_new, v_new, seq_lens, s)) != RK_OK) return rc;
        const int64_t w_stride = pooled_row_stride(max_rows);
        rc = full_attn_stage(geom, q, state.cache, state.n_attend, max_rows, out, ws.scores, w_stride, nullptr,
                             nullptr, 0, ws, s, false, -1, false, RK_AGG_MAX, false, nch);
        if (rc != RK_OK) return rc;
        return update_stage(geom, state, ws.scores, w_stride, max_rows, budget, recent, agg, dropped, s);
    }
    if ((rc = h2o_attn_stage(geom, q, state, k_new, v_new, budget, ws, s)) != RK_OK) return rc;
    const int32_t* counters = ragged_batch_of(geom) != 0 ? ws.counters : nullptr;
    switch (geom->n_q_heads / geom->n_kv_heads) {
#define RK_CASE(g) case g: hipLaunchKernelGGL((h2o_finish_kernel<g>), dim3(geom->n_kv_heads, geom->batch), dim3(kH2oThreads), 0, s, state, \
                       ws.scores, pooled_row_stride(max_rows), ws.part_ml, ws.part_o, ws.max_chunks, nch, counters, max_rows, \
                       (const uint16_t*)k_new, (const uint16_t*)v_new, seq_lens, geom->n_kv_heads, budget, recent, agg, \
                       (uint16_t*)out, dropped, state.cache.capacity); break;
        RK_CASE(1) RK_CASE(2) RK_CASE(3) RK_CASE(4) RK_CASE(5) RK_CASE(6) RK_CASE(7) RK_CASE(8)
#undef RK_CASE
        default: return RK_ERR_UNSUPPORTED;
    }
    return launch_status();
}
