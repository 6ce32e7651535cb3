// Shared by the attention kernels: their parameters, the arguments that arrive in registers, loads of cache rows.
#pragma once

#include "rk_internal.h"
#include "rk_device.h"

namespace rk {

struct AttnParams {
    const uint16_t* q;                 // bf16 [B, Hq, 128]
    const uint16_t* k1; const uint16_t* v1; int64_t s1_b, s1_h;   // small cache (TWO_SEG only)
    const uint16_t* k2; const uint16_t* v2; int64_t s2_b, s2_h;   // full cache
    const int32_t* tail_start;         // TWO_SEG only
    const int32_t* seq_lens;
    int32_t n_sel;                     // rows taken from the small cache (TWO_SEG only)
    int32_t evict;                     // ... less one per row decoded since the refresh (fixed-size small cache)
    int32_t tail_wg;                   // TWO_SEG: the rows of the full cache have a workgroup of their own (grid x = nch + 1)
    int32_t max_rows2;                 // host bound on the rows taken from the full cache
    int32_t cap1, cap2;                // rows allocated in the small / full cache
    int32_t nch;                       // workgroups per (sequence, KV head): the launch's grid x
    int32_t Hq, Hkv;
    float scale;
    uint16_t* out;                     // bf16 [B, Hq, 128]
    float* weights; int64_t w_stride;  // raw scores go here first (EMIT only)
    int32_t w_vec;                     // rows of `weights` start 16-byte aligned: vector stores allowed
    int32_t w_inter;                   // groups of 4 heads, scores kept in the workspace: the 4 heads of a position side by side
                                       // (score of head gi at position j of group (b, g): weights[(b*Hq + g*4) * w_stride + 4*j + gi])
    float* lse;                        // fp32 [B, Hq], never NULL here
    const int32_t* pred; int32_t pred_val;
    int32_t* counters; float* part_ml; float* part_o; int32_t max_chunks;
    uint32_t* epochs; uint32_t* tag_rows;     // TAGGED only: call number per (sequence, KV head), tagged partial results
    const int32_t* idx; int32_t idx_stride;   // LAZY only: the selection [B, Hkv, idx_stride] whose rows are not gathered yet
    float* trig_q_ref; float* trig_sim; int32_t* trig_need; float trig_threshold;   // TRIG only: the query-similarity test
    int32_t tail_inside;               // two_tile_form only: the rows since follow the small cache's in its workgroups
    int32_t* mark_tail; int32_t* mark_count;  // the gather inside the step only: tail_start <- seq_lens, refreshes counted (may be NULL)
    int32_t ragged_batch;              // != 0 (= batch): workgroups are shared out by length, see ragged_share_lane
    int32_t share_cap;                 // ... at most this many to a sequence
    int32_t* n_attend;                 // APPEND only: [B], rows attended over, for the kernel that follows
    int32_t slice_merge;               // TAGGED: every workgroup merges a slice of the output (all workgroups of the launch are resident together)
    int32_t slice_spin;                // ... re-reading rows still in flight at most this often before it leaves its slice to the last one
};

// The partial step in one tile per workgroup (rk_partial.hip): `waves` wavefronts of 16 rows.
// idx given: the gather inside the step.
__attribute__((visibility("hidden")))
int launch_partial_tile(const AttnParams& p, int batch, int G, const TileForm& form, bool trig, const int32_t* idx, hipStream_t st);

constexpr int kSplitWaves = 4, kTileRows = 32;
constexpr int kNoTailWg = 0xff;                   // top byte of the kernel argument s_b_and_tail: no workgroup for the tail rows
constexpr int kHeadsFirst = 0xfe;                 // ... (launches over the full cache only) grid x = KV head, y = sequence, z = chunk

// All global stores this thread issued so far are acknowledged once this returns.
__device__ __forceinline__ void wait_stores_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// ds_read_b64_tr_b16: every 16 lanes hand in 16 addresses of 4 consecutive bf16 (a 16 x 4
// matrix M, row = lane) and lane i gets back M[i/4 + 4e][i%4] for e = 0..3.
typedef short v4s __attribute__((ext_vector_type(4)));
typedef short v8s __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));      // 16 bytes in four registers
// 16-byte load of cache rows.  STREAM: the rows are read once per step and not again before
// far more than the caches hold has passed through (the full cache): a non-temporal load, which
// leaves the L2 and the last-level cache to the data that does come back (the small caches, read
// at every partial step).  Measured: the kernel that streams K and V of the full cache runs 4%
// faster with it, the scores-only pass too where its keys outgrow the last-level cache (kScoreStreamBytes; below
// it is 3-5% slower); the partial step is 3% slower.
template <bool STREAM>
__device__ __forceinline__ u32x4 load_rows16(const uint16_t* p) {
    if (STREAM) return __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
    return *reinterpret_cast<const u32x4*>(p);
}
__device__ __forceinline__ v4s lds_read_tr16(const uint16_t* ptr) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s*)ptr);
}
// Two fp32 -> packed bf16 pair, round to nearest even (v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    const f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
constexpr int kTagSpinLimit = 1 << 16;            // re-reads of rows still in flight before giving up (NaN output)
constexpr int kAgentScopeAux = 16;                // cache-policy operand of buffer loads and stores: sc1

// ---- partial results as rows of two output dims ----
// The partial result of one workgroup (a chunk of the rows) is, per head, 64 rows of 16 bytes, dims 2r and 2r + 1 each:
// { x[2r], x[2r+1], lambda, tag } with x the chunk's own normalised output, lambda = m + log2 l its log-sum-exp in units of
// ln 2 and tag the number of the call.  A row is one 16-byte store of one lane and one 16-byte load of one lane, never split: a row whose
// tag is this call's holds this call's values.  Every row carries the lambda that weighs it,
//   Lambda = max_c lambda_c,  w_c = 2^{lambda_c - Lambda},  out = sum_c w_c x_c / sum_c w_c,
// so a lane has all it needs in the rows it reads.  (The other tagged form, three dims to a row and lambda in a row of its
// own, keeps its tags in the same word of rows on the same 16-byte grid of the same region: neither can take a row of
// the other for one of this call's.)
//
// EXACT: a lambda of fp32 puts ln 2 ulp(lambda) / 2 into a weight (2e-5 at scores of 400, 1.7e-4 at 4096).  Launches whose
// shapes took (max, sum) pairs before this form did keep them: the rows hold the sums 2^{s - m} v as they are, { x, x, m, tag }, and one more row
// per head, behind all partial results (head by head: a merge reads neighbours), holds { l, -, m, tag }; w_c = 2^{m_c - max m}, out = sum_c w_c x_c / sum_c w_c l_c.
//
// The merge is cut into units of U consecutive rows of a head, a wavefront each, 64 / U lanes to a row: lane U q + i
// sums the chunks q, q + 64/U, q + 2 * 64/U, ... (at most TB) of row i, and the sums are added across the lanes in a fixed
// order.  Which workgroup merges a unit does not change a bit of it.
constexpr int kPairRows = kD / 2;                 // rows of a head
// log2 U for a number of partial results: about five rows for a lane to read, at most 64 units (a bit each).
template <int G> __device__ __forceinline__ int pair_unit_shift(int nchunks) { return nchunks <= 20 ? 4 : (nchunks <= 40 || G > 4) ? 3 : 2; }
// What a lane reads of a unit: the first partial result's number, the row, and the two's place in the region.  EXACT: and the row of l of
// one partial result (a unit lies within a head), the lane's number, so that the sum of the weights is one of all lanes.
template <int G, bool EXACT> struct PairLane {
    static constexpr int STRIDE = G * kPairRows * 16;              // bytes of a partial result
    int q, row, first, last, sum;
    __device__ __forceinline__ PairLane(int unit, int shift, int nchunks) {
        const int lane = threadIdx.x & 63;
        q = lane >> shift;
        row = (unit << shift) + (lane & ((1 << shift) - 1));       // of all the group's rows
        first = q * STRIDE + row * 16;
        last = (nchunks - 1) * STRIDE + row * 16;
        if (EXACT) sum = sum_row(row / kPairRows, min(lane, nchunks - 1));
    }
    static __device__ __forceinline__ int sum_row(int head, int c) { return kTileExactChunks * STRIDE + (head * kTileExactChunks + c) * 16; }
};

// Max and sum over the lanes i, i + U, i + 2U ... of the wavefront.
template <int U>
__device__ __forceinline__ float lanes_max(float v) {
    if (U <= 8) v = fmaxf(v, dpp_move_f<kDppRor8>(v));
    if (U <= 4) v = fmaxf(v, dpp_move_f<kDppRor4>(v));
    if (U <= 2) v = fmaxf(v, dpp_move_f<kDppXor2>(v));
    if (U <= 1) v = fmaxf(v, dpp_move_f<kDppXor1>(v));
    return max_xor32(max_xor16(v));
}
template <int U>
__device__ __forceinline__ float lanes_sum(float v) {
    if (U <= 8) v += dpp_move_f<kDppRor8>(v);
    if (U <= 4) v += dpp_move_f<kDppRor4>(v);
    if (U <= 2) v += dpp_move_f<kDppXor2>(v);
    if (U <= 1) v += dpp_move_f<kDppXor1>(v);
    return sum_xor32(sum_xor16(v));
}

// One unit.  Rows still in flight are re-read at most `spin` times; if some are still missing then, the output is left
// alone and the result is false (final: NaN is written instead).  `out`: the group's first head.
template <int G, bool EXACT, int U, int TB>
__device__ __forceinline__ bool merge_pair_unit(uint16_t* out, const __amdgpu_buffer_rsrc_t rsrc, const PairLane<G, EXACT> at, int nchunks,
                                                uint32_t tag, int spin, bool final) {
    constexpr int LPR = 64 / U;
    u32x4 v[TB], l;
    bool ok = false;
    int tries = 0;
    while (!__all(ok) && tries++ < spin) {
        if (tries > 1) __builtin_amdgcn_s_sleep(2);
#pragma unroll
        for (int u = 0; u < TB; ++u)
            v[u] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, min(at.first + u * LPR * PairLane<G, EXACT>::STRIDE, at.last), 0, kAgentScopeAux);
        if constexpr (EXACT) l = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at.sum, 0, kAgentScopeAux);
        uint32_t bad = 0;
#pragma unroll
        for (int u = 0; u < TB; ++u) bad |= v[u].w ^ tag;
        if constexpr (EXACT) bad |= l.w ^ tag;
        ok = bad == 0u;
    }
    const bool good = __all(ok);
    if (!good && !final) return false;
    float lam[TB], ref = -3.0e38f;                                 // finite: exponents below are never inf - inf
#pragma unroll
    for (int u = 0; u < TB; ++u) {
        lam[u] = at.q + u * LPR < nchunks ? __uint_as_float(v[u].z) : -INFINITY;
        ref = fmaxf(ref, lam[u]);
    }
    const int lane = threadIdx.x & 63;
    if constexpr (EXACT) ref = fmaxf(ref, lane < nchunks ? __uint_as_float(l.z) : -INFINITY);
    ref = lanes_max<EXACT ? 1 : U>(ref);
    float a0 = 0.f, a1 = 0.f, den = 0.f;
#pragma unroll
    for (int u = 0; u < TB; ++u) {
        const float wu = fast_exp2(lam[u] - ref);                  // 0 beyond nchunks and for empty chunks
        a0 = fmaf(wu, __uint_as_float(v[u].x), a0);
        a1 = fmaf(wu, __uint_as_float(v[u].y), a1);
        if constexpr (!EXACT) den += wu;
    }
    if constexpr (EXACT) den = lane < nchunks ? fast_exp2(__uint_as_float(l.z) - ref) * __uint_as_float(l.x) : 0.f;
    a0 = lanes_sum<U>(a0); a1 = lanes_sum<U>(a1); den = lanes_sum<EXACT ? 1 : U>(den);
    const float inv = den > 0.f ? __builtin_amdgcn_rcpf(den) : 0.f;
    const float nan = __uint_as_float(0x7fc00000u);
    const uint32_t pair = good ? pack_bf16(a0 * inv, a1 * inv) : pack_bf16(nan, nan);
    if (at.q == 0) {                                               // (out is 2-byte aligned)
        uint16_t* o = out + 2 * at.row;
        o[0] = (uint16_t)pair; o[1] = (uint16_t)(pair >> 16);
    }
    return true;
}
template <int G, bool EXACT>
__device__ __forceinline__ bool merge_pairs(uint16_t* out, const __amdgpu_buffer_rsrc_t rsrc, const PairLane<G, EXACT> at, int nchunks,
                                            uint32_t tag, int spin, bool final) {
    if (nchunks <= 8) return merge_pair_unit<G, EXACT, 16, 2>(out, rsrc, at, nchunks, tag, spin, final);
    if (nchunks <= 20) return merge_pair_unit<G, EXACT, 16, 5>(out, rsrc, at, nchunks, tag, spin, final);
    if (nchunks <= 40) return merge_pair_unit<G, EXACT, 8, 5>(out, rsrc, at, nchunks, tag, spin, final);
    if constexpr (G <= 4) return merge_pair_unit<G, EXACT, 4, 5>(out, rsrc, at, nchunks, tag, spin, final);
    else                  return merge_pair_unit<G, EXACT, 8, 9>(out, rsrc, at, nchunks, tag, spin, final);
}

}  // namespace rk
