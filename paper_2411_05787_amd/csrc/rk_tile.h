// One workgroup's part of the partial step in one tile (rk_partial.hip says what it is made for), shared with the launch that holds
// a test step's two branches (rk_attn.hip).
#pragma once

#include "rk_attn_common.h"

namespace rk {

// What the kernel needs beyond its preloaded arguments, in the order in which it needs it.
struct TileParams {
    float scale2;                             // scale * log2 e: scores, maxima and lambda are kept in units of ln 2
    int32_t n_sel, evict, max_rows2, cap1, cap2, slice_spin, pred_val;
    uint32_t* epochs; uint16_t* out; int32_t* counters; uint32_t* tag_rows;
    const uint16_t* k2; const uint16_t* v2; int64_t s2_b, s2_h;
    const int32_t* pred; float* trig_q_ref;
    union { float* trig_sim; int32_t* mark_count; };      // GATHER: refreshes counted (may be NULL), tail_start (three lines of 64 bytes of arguments, not four)
    union { int32_t* trig_need; int32_t* mark_tail; };
    float trig_threshold;
};
// Preloaded argument `rows_heads`: rows of the small cache that exist whatever the lengths say | a predicate is given | KV heads << 16.
constexpr int kSpecBits = 15, kPredBit = 1 << kSpecBits;
constexpr int kTailInside = 0x80;             // in the top byte of `s_b_and_tail`, beside the first workgroup with rows of the full cache
static_assert(kMergeChunks < kTailInside, "workgroups of the small cache");
static_assert(kMergeChunks * 256 < (1 << kSpecBits), "rows of the small cache");

// LDS that the parts of a kernel use one after the other (ROOM bytes; 0: a part has its own).
template <int BYTES> __device__ __forceinline__ unsigned char* lds_room() {
    __shared__ __attribute__((aligned(16))) unsigned char room[BYTES];
    return room;
}

// Attention over the small cache and the rows decoded since the refresh, where no workgroup has more rows than it holds
// at once: 16 per wavefront.  Workgroup c of KV head g of sequence b.  With the trigger's test: true in the wavefronts with rows if the
// sequence needs a full step, and nothing has been published then.
// GATHER: the step right after a selection, with the gather in it.  The rows of the small cache come from the full one (k2 / v2) through the
// selection, which takes tail_start's place among the arguments, and are written to the small cache (k1 / v1) on the way, those beyond the
// sequence's end too; a row whose entry is no position of the full cache is the small cache's own.  No rows since.
enum TestBy { kNoTest, kTestBeside, kTestInside };      // the test is the work of a wavefront more, or of the first one with rows
// R: tiles of 16 rows to a wavefront.  Two: 32 rows next to each other, requested at once; or (LATE) the first tiles of all workgroups have the first half
// of the small cache and the second ones, requested as soon as the lengths are known, the other half: a cache with few rows is read for what it holds, and by
// every workgroup.  Where the launch has no workgroups for the rows since, they follow those of the small cache in the slots that are left
// (kTailInside); the host knows that they fit.
template <int G, int NW, TestBy TEST, bool EXACT, bool GATHER = false, int R = 1, int ROOM = 0, bool LATE = false>
__device__ __forceinline__
bool partial_tile(const uint16_t* k1, const uint16_t* v1, int64_t s_b_and_tail, int32_t s_h, uint32_t rows_heads,
                  const int32_t* seq_lens, const int32_t* tail_start, const uint16_t* q, const TileParams& p, int c, int g, int b) {
    constexpr bool TRIG = TEST != kNoTest;
    constexpr int WG = 16 * NW * R;           // rows of a workgroup
    constexpr int STEP = LATE ? 16 * NW : WG; // rows from a workgroup's first to the next one's
    constexpr int DT = 8 / NW, KS = NW * R / 2;   // P V: tiles of 16 dims of a wavefront, steps of 32 rows
    static_assert(R == 1 || !GATHER, "not built");
    static_assert(!LATE || (R == 2 && !TRIG), "two tiles, no test");
    // P's lanes in LDS: those beyond the group hold nothing that is used, so where there is much of it they read the others'
    constexpr int GP = R == 1 ? 16 : G <= 4 ? 4 : 8;
    constexpr int VS = kD + 8;                // LDS row stride of the V tile (272 bytes: rows spread over banks)
    const int64_t s_b = s_b_and_tail & ((1ll << 56) - 1);
    const int first_tail = (int)(s_b_and_tail >> 56) & (R > 1 ? kTailInside - 1 : 0xff);      // workgroups from here on have rows of the full cache, those before of the small one
    const bool inside = R > 1 && (s_b_and_tail >> 56 & kTailInside) != 0;
    const int spec_rows = rows_heads & ((1 << kSpecBits) - 1), n_kv = rows_heads >> 16;
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n16 = lane & 15, c4 = lane >> 4;
    const int64_t bg = (int64_t)b * n_kv + g;
    if (!TRIG && (rows_heads & kPredBit) != 0 && p.pred[b] != p.pred_val) return false;
    // ---- the scalars of the whole kernel are requested here, in one round trip (left to itself the compiler reads them
    //      where they are used, a round trip each), and waited for behind the requests for the first rows ----
    static_assert(!GATHER || !TRIG, "no test right after a selection");
    const int len_raw = seq_lens[b], tail_raw = GATHER ? len_raw : tail_start[b];
    const float scale2 = p.scale2;
    const int spin = p.slice_spin, n_sel = p.n_sel, evict = p.evict, max_rows2 = p.max_rows2, cap1 = p.cap1,
              cap2 = p.cap2;
    uint16_t* const out_all = p.out;
    int32_t* const counters = p.counters;
    uint32_t* const tag_rows = p.tag_rows;
    uint32_t* const epochs = p.epochs;
    const uint16_t* const k2 = p.k2;
    const uint16_t* const v2 = p.v2;
    const int64_t s2_b = p.s2_b, s2_h = p.s2_h;
    __builtin_amdgcn_sched_barrier(0);
    SimLoads ld;                              // kTestInside: the first requests, so that the test is worked out while the rows are on their way
    if constexpr (TEST == kTestInside)
        if (w == 0) similarity_request(q, p.trig_q_ref, b, n_kv * G, ld);
    // ---- K rows, queries and V rows of a workgroup of the small cache, requested before any length is known: the rows of a
    //      cache are a buffer, whose rows past the end read as zero ----
    u32x4 kA[R][4], vA[R][4], qa[4];
    k1 += (uint64_t)s_b * (uint32_t)b + (uint64_t)(uint32_t)s_h * (uint32_t)g;
    v1 += (uint64_t)s_b * (uint32_t)b + (uint64_t)(uint32_t)s_h * (uint32_t)g;
    const int k_lane = n16 * (kD * 2) + c4 * 16, v_lane = c4 * (kD * 2) + n16 * 16;      // bytes, from the wavefront's first row
    auto request_k = [&](const uint16_t* k, int rows, int row) {
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(k), 0, rows * (kD * 2), 0x00020000);
#pragma unroll
        for (int x = 0; x < 4 * R; ++x)
            kA[x >> 2][x & 3] = __builtin_amdgcn_raw_buffer_load_b128(rk, (row + (x >> 2) * 16) * (kD * 2) + k_lane + (x & 3) * 64, 0, 0);
    };
    auto request_v = [&](const uint16_t* v, int rows, int row) {
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(v), 0, rows * (kD * 2), 0x00020000);
#pragma unroll
        for (int x = 0; x < 4 * R; ++x)
            vA[x >> 2][x & 3] = __builtin_amdgcn_raw_buffer_load_b128(rv, row * (kD * 2) + v_lane + x * 4 * (kD * 2), 0, 0);
    };
    auto request_tile = [&](const uint16_t* k, const uint16_t* v, int rows, int row, int x) {
        const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(k), 0, rows * (kD * 2), 0x00020000);
        const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(v), 0, rows * (kD * 2), 0x00020000);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) kA[x][kk] = __builtin_amdgcn_raw_buffer_load_b128(rk, row * (kD * 2) + k_lane + kk * 64, 0, 0);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) vA[x][jj] = __builtin_amdgcn_raw_buffer_load_b128(rv, row * (kD * 2) + v_lane + jj * 4 * (kD * 2), 0, 0);
    };
    int r_first = c * STEP + w * (LATE ? 16 : 16 * R), step = LATE ? first_tail * STEP : 16;      // the wavefront's first row, rows to its next tile's
    // (inside: the last workgroup, which has the most of the rows since, requests nothing yet: it waits for the lengths and requests every row from
    // where it is; requested once more, those rows would come behind everybody's)
    const bool waits = !LATE && inside && c + 1 == first_tail;
    const int early = c < first_tail && !waits ? spec_rows : 0;
    // GATHER: where the rows of this lane are: row n16 of the wavefront's 16 for K, rows 4 jj + c4 for V
    int from_k = -1, from_v[4] = {-1, -1, -1, -1};
    if constexpr (GATHER) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<int32_t*>(tail_start) + bg * spec_rows, 0, spec_rows * 4, 0x00020000);
        from_k = (int)__builtin_amdgcn_raw_buffer_load_b32(rs, (r_first + n16) * 4, 0, 0);
    } else if constexpr (!LATE) {
        request_k(k1, early, r_first);
    }
    {                                         // (heads beyond the group read as zero)
        const __amdgpu_buffer_rsrc_t rq = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(q) + bg * G * kD, 0, G * kD * 2, 0x00020000);
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) qa[kk] = __builtin_amdgcn_raw_buffer_load_b128(rq, k_lane + kk * 64, 0, 0);
    }
    if constexpr (LATE) request_tile(k1, v1, early, r_first, 0);
    else if constexpr (!GATHER) request_v(v1, early, r_first);
    asm volatile("" :: "s"(scale2), "s"(spin), "s"(out_all), "s"(counters), "s"(tag_rows), "s"(epochs),
                 "s"(k2), "s"(v2), "s"(s2_b), "s"(s2_h), "s"(p.pred_val));
    const uint32_t epoch = *(const __attribute__((address_space(4))) uint32_t*)(epochs + bg);      // (the kernel's own store comes after: a scalar load)
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (GATHER) {
        from_k = r_first + n16 < spec_rows && (uint32_t)from_k < (uint32_t)cap2 ? from_k : -1;
        const uint64_t at = (uint64_t)s2_b * (uint32_t)b + (uint64_t)s2_h * (uint32_t)g;
        auto row_at = [&](const uint16_t* full, const uint16_t* small, int from, int r) {
            return from >= 0 ? full + at + (int64_t)from * kD : small + (int64_t)min(r, spec_rows - 1) * kD;
        };
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            from_v[jj] = __shfl(from_k, jj * 4 + c4);
            kA[0][jj] = *reinterpret_cast<const u32x4*>(row_at(k2, k1, from_v[jj], r_first + jj * 4 + c4) + n16 * 8);
        }
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) vA[0][jj] = *reinterpret_cast<const u32x4*>(row_at(v2, v1, from_v[jj], r_first + jj * 4 + c4) + n16 * 8);
        if (c == 0 && g == 0 && tid == 0) {
            if (p.mark_tail != nullptr) p.mark_tail[b] = len_raw;
            if (p.mark_count != nullptr) p.mark_count[b] += 1;      // (one writer per sequence and launch)
        }
    }
    auto write_rows = [&](const uint16_t* small, const u32x4 (&rows)[4]) {
        if constexpr (GATHER) {
            uint16_t* to = const_cast<uint16_t*>(small) + (int64_t)(r_first + c4) * kD + n16 * 8;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
                if (from_v[jj] >= 0) *reinterpret_cast<u32x4*>(to + jj * 4 * kD) = rows[jj];
        }
    };

    __shared__ __attribute__((aligned(16))) uint16_t own[ROOM ? 1 : WG][VS];
    uint16_t (*sV)[VS] = own;
    if constexpr (ROOM != 0) {
        static_assert(ROOM >= (int)(WG * VS * sizeof(uint16_t)), "room");
        sV = reinterpret_cast<uint16_t (*)[VS]>(lds_room<ROOM>());
    }
    __shared__ __attribute__((aligned(16))) uint2 sP[2][KS][4 * GP][2];  // hi and lo, step, lane, half of the step
    __shared__ __attribute__((aligned(16))) float sM[16][NW], sL[16][NW];
    __shared__ int sTicket, sNeed;
    __shared__ unsigned long long sPend;

    // The test.  The wavefronts with rows learn the decision with the maxima.  Where the sequence needs a full step every workgroup has
    // read the old reference by the time it takes its ticket (the second word of the sequence's first counter line: zero
    // between launches); the last one stores the new one.
    float qbar[8];
    auto test = [&]() {
        const float s = similarity_finish(q, b, n_kv * G, ld, qbar);
        const bool need = !(s > p.trig_threshold);
        if (lane == 0) {
            sNeed = need ? 1 : 0;
            if (c == 0 && g == 0) { p.trig_sim[b] = s; p.trig_need[b] = need ? 1 : 0; }
        }
        return need;
    };
    auto new_reference = [&]() {
        int last = 0;
        if (lane == 0) {
            int32_t* ticket = counters + (int64_t)b * n_kv * kCounterStride + 1;
            const int seen = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            last = seen == (int)(gridDim.x * gridDim.y) - 1 ? 1 : 0;
            if (last) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        last = __builtin_amdgcn_readfirstlane(last);
        if (last && lane < 16) {
            float4* rp = reinterpret_cast<float4*>(p.trig_q_ref + (int64_t)b * kD + lane * 8);
            rp[0] = make_float4(qbar[0], qbar[1], qbar[2], qbar[3]);
            rp[1] = make_float4(qbar[4], qbar[5], qbar[6], qbar[7]);
        }
    };
    if constexpr (TEST == kTestBeside) {
        if (w == NW) {
            similarity_request(q, p.trig_q_ref, b, n_kv * G, ld);
            const bool need = test();
            lds_barrier();
            if (need) new_reference();
            return false;
        }
    }
    if constexpr (TEST == kTestInside)
        if (w == 0) test();
    // the decision, once every wavefront has what it brings to the first barrier
    auto needs_full = [&]() {
        const bool need = sNeed != 0;
        if constexpr (TEST == kTestInside)
            if (need && w == 0) new_reference();
        return need;
    };

    // ---- the row list of this (sequence, KV head) (lengths clamped to the allocated rows: no access leaves the caches) ----
    const int len = min(len_raw, cap2), t0 = min(max(tail_raw, 0), cap2), recent = max(len - t0, 0);
    // fixed-size small cache: every row decoded since the refresh pushed out the selected row with the lowest score (the last)
    int keep = max(n_sel - (evict != 0 ? recent : 0), 0);
    keep = min(keep, cap1);
    asm("" : "+s"(keep));                     // (scalar minima, one after the other)
    const int n1 = min(keep, t0), n2 = min(recent, max_rows2);
    // partial results in all (an empty sequence leaves one of no rows), this workgroup's place among them, the end of its rows
    const int n_in = inside ? n2 : 0;         // rows since in the slots behind the small cache's
    const int n_late = min((int)((uint32_t)(n1 + n_in + 16 * NW - 1) / (16 * NW)), first_tail);      // LATE: workgroups whose first tiles have rows
    const int n_main = LATE ? max(n_late, inside || n2 == 0 ? 1 : 0) : inside ? max((int)((uint32_t)(n1 + n2 + WG - 1) / WG), 1) : first_tail != 0 ? max((int)((uint32_t)(n1 + WG - 1) / WG), n2 == 0 ? 1 : 0) : 0;
    const int n_tail = inside ? 0 : max((int)((uint32_t)(n2 + WG - 1) / WG), first_tail != 0 ? 0 : 1);
    const int nchunks = n_main + n_tail;
    const bool tail = c >= first_tail;
    const int c_rec = tail ? c - first_tail + n_main : c, row1 = tail ? n1 + n2 : n1 + n_in;
    if (c_rec >= (tail ? nchunks : n_main)) {
        if constexpr (TRIG) {                   // (the wavefront with the test waits for everybody)
            lds_barrier();
            return needs_full();
        }
        write_rows(k1, kA[0]);
        write_rows(v1, vA[0]);
        return false;
    }
    if (tail) {
        // row r of the list lives at row t0 + r - n1 of the full cache
        if constexpr (LATE) {
            r_first = n1 + (c - first_tail) * WG + w * 16 * R;
            step = 16;
        } else {
            r_first += n1 - first_tail * WG;
        }
        const uint64_t at = (uint64_t)s2_b * (uint32_t)b + (uint64_t)s2_h * (uint32_t)g + (uint64_t)(uint32_t)t0 * kD;
        request_k(k2 + at, n2, r_first - n1);
        request_v(v2 + at, n2, r_first - n1);
    }
    if constexpr (LATE) {
        if (!tail) {
            // a tile with rows since (the same for the whole wavefront): row r of the list is the small cache's, or row t0 + r - n1 of the full one; past
            // the list's end its last row again (masked)
            const uint64_t at = (uint64_t)s2_b * (uint32_t)b + (uint64_t)s2_h * (uint32_t)g;
            auto request_list = [&](int x) {
                auto row_at = [&](const uint16_t* small, const uint16_t* full, int r) {
                    r = min(r_first + x * step + r, row1 - 1);
                    return r < n1 ? small + (int64_t)r * kD : full + at + (int64_t)(t0 + r - n1) * kD;
                };
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) kA[x][kk] = *reinterpret_cast<const u32x4*>(row_at(k1, k2, n16) + c4 * 8 + kk * 32);
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) vA[x][jj] = *reinterpret_cast<const u32x4*>(row_at(v1, v2, jj * 4 + c4) + n16 * 8);
            };
            auto has_since = [&](int x) { return inside && n2 > 0 && r_first + x * step < row1 && r_first + x * step + 16 > n1; };
            if (has_since(0)) request_list(0);
            if (has_since(1)) request_list(1);
            else request_tile(k1, v1, n1, r_first + step, 1);
        }
    } else if constexpr (R > 1) {
        if (waits || (inside && n2 > 0 && r_first < row1 && r_first + 16 * R > n1)) {      // (the same for the whole wavefront)
            // row r of the list: the small cache's, or row t0 + r - n1 of the full one; past the list's end its last row again (masked)
            const uint64_t at = (uint64_t)s2_b * (uint32_t)b + (uint64_t)s2_h * (uint32_t)g;
            auto row_at = [&](const uint16_t* small, const uint16_t* full, int r) {
                r = max(min(r, row1 - 1), 0);
                return r < n1 || row1 == 0 ? small + (int64_t)r * kD : full + at + (int64_t)(t0 + r - n1) * kD;
            };
#pragma unroll
            for (int x = 0; x < 4 * R; ++x)
                kA[x >> 2][x & 3] = *reinterpret_cast<const u32x4*>(row_at(k1, k2, r_first + (x >> 2) * 16 + n16) + c4 * 8 + (x & 3) * 32);
#pragma unroll
            for (int x = 0; x < 4 * R; ++x)
                vA[x >> 2][x & 3] = *reinterpret_cast<const u32x4*>(row_at(v1, v2, r_first + x * 4 + c4) + n16 * 8);
        }
    }
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(tag_rows + bg * kTagRegionRows * G * 4, 0,
                                                                          kTagRegionRows * G * 16, 0x00020000);
    const uint32_t tag = max(epoch + 1u, 1u);                          // this call's number: never 0
    // this wavefront's first unit of the merge, worked out while the rows are on their way
    const int shift = pair_unit_shift<G>(nchunks), units = (kPairRows * G) >> shift, unit0 = c_rec + (NW - 1 - w) * nchunks;
    PairLane<G, EXACT> at0(unit0, shift, nchunks);
    asm volatile("" : "+v"(at0.q), "+v"(at0.row), "+v"(at0.first), "+v"(at0.last) : "s"(tag));
    if constexpr (EXACT) asm volatile("" : "+v"(at0.sum));

    if constexpr (GATHER) {                   // whole rows of K, into the operand layout by way of the V tile's room
        write_rows(k1, kA[0]);
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) *reinterpret_cast<u32x4*>(&sV[w * 16 + jj * 4 + c4][n16 * 8]) = kA[0][jj];
        wave_lds_sync();
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) kA[0][kk] = *reinterpret_cast<const u32x4*>(&sV[w * 16 + n16][kk * 32 + c4 * 8]);
        wave_lds_sync();
    }
    // ---- S^T = K Q^T: head n16, rows 4 c4 + i of each of the wavefront's tiles ----
    float s[R][4];
    const bool whole = r_first + (LATE ? step + 16 : 16 * R) <= row1;
#pragma unroll
    for (int x = 0; x < R; ++x) {
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kA[x][kk]), __builtin_bit_cast(bf16x8, qa[kk]), acc, 0, 0, 0);
#pragma unroll
        for (int i = 0; i < 4; ++i) s[x][i] = acc[i] * scale2;
        if (!whole) {
#pragma unroll
            for (int i = 0; i < 4; ++i) s[x][i] = r_first + x * step + 4 * c4 + i < row1 ? s[x][i] : -INFINITY;
        }
    }
    float mx = fmaxf(fmaxf(s[0][0], s[0][1]), fmaxf(s[0][2], s[0][3]));
#pragma unroll
    for (int x = 1; x < R; ++x) mx = fmaxf(mx, fmaxf(fmaxf(s[x][0], s[x][1]), fmaxf(s[x][2], s[x][3])));
    mx = max_xor32(max_xor16(mx));
    if (c4 == 0) sM[n16][w] = mx;
    lds_barrier();
    if constexpr (TRIG) {
        if (needs_full()) return true;
    }
    // ---- P against the workgroup's maximum, as two bf16 operands hi + lo (to about 2^-17) ----
    float M = sM[n16][0];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) M = fmaxf(M, sM[n16][ww]);
    const float ref = M == -INFINITY ? 0.f : M;
    const int p_lane = GP == 16 ? lane : c4 * GP + (n16 & (GP - 1));
    float ps = 0.f;
#pragma unroll
    for (int x = 0; x < R; ++x) {
        float pr[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) { pr[i] = fast_exp2(s[x][i] - ref); ps += pr[i]; }
        const uint2 hi = make_uint2(pack_bf16(pr[0], pr[1]), pack_bf16(pr[2], pr[3]));
        const uint2 lo = make_uint2(pack_bf16(pr[0] - bf16_lo(hi.x), pr[1] - bf16_hi(hi.x)),
                                    pack_bf16(pr[2] - bf16_lo(hi.y), pr[3] - bf16_hi(hi.y)));
        const int at = w * R + x;
        if (GP == 16 || n16 < GP) {
            sP[0][at >> 1][p_lane][at & 1] = hi;
            sP[1][at >> 1][p_lane][at & 1] = lo;
        }
    }
    __builtin_amdgcn_sched_barrier(0);        // (P is on its way before the sums are worked out)
    ps = sum_xor32(sum_xor16(ps));
    if (c4 == 0) sL[n16][w] = ps;
    write_rows(v1, vA[0]);
    if (!whole) {       // V rows past the end hold whatever the cache holds there, maybe NaN: P is 0 for them, but 0 * NaN is NaN
#pragma unroll
        for (int x = 0; x < 4 * R; ++x)
            if (r_first + (LATE ? (x >> 2) * step + (x & 3) * 4 : x * 4) + c4 >= row1) vA[x >> 2][x & 3] = u32x4{0u, 0u, 0u, 0u};
    }
#pragma unroll
    for (int x = 0; x < 4 * R; ++x) *reinterpret_cast<u32x4*>(&sV[w * 16 * R + x * 4 + c4][n16 * 8]) = vA[x >> 2][x & 3];
    lds_barrier();
    // ---- O^T = V^T P^T of all the workgroup's rows: this wavefront's dims, head n16, four consecutive dims per lane ----
    float L = sL[n16][0];
#pragma unroll
    for (int ww = 1; ww < NW; ++ww) L += sL[n16][ww];
    f32x4 o[DT][2];
#pragma unroll
    for (int t = 0; t < DT; ++t) { o[t][0] = f32x4{0.f, 0.f, 0.f, 0.f}; o[t][1] = f32x4{0.f, 0.f, 0.f, 0.f}; }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        const bf16x8 p_hi = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&sP[0][ks][p_lane][0]));
        const bf16x8 p_lo = __builtin_bit_cast(bf16x8, *reinterpret_cast<const uint4*>(&sP[1][ks][p_lane][0]));
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            const uint16_t* vsrc = &sV[32 * ks + 4 * c4 + (n16 >> 2)][(w * DT + t) * 16 + 4 * (n16 & 3)];
            const v4s v0 = lds_read_tr16(vsrc), v1 = lds_read_tr16(vsrc + 16 * VS);
            const bf16x8 vb = __builtin_bit_cast(bf16x8, __builtin_shufflevector(v0, v1, 0, 1, 2, 3, 4, 5, 6, 7));
            o[t][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb, p_hi, o[t][0], 0, 0, 0);
            o[t][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vb, p_lo, o[t][1], 0, 0, 0);
        }
    }
    float inv = 1.f, lam = M;                 // EXACT: the sums as they are, weighed by their maximum (-inf: no rows)
    if constexpr (!EXACT) {
        inv = L > 0.f ? __builtin_amdgcn_rcpf(L) : 0.f; lam = L > 0.f ? M + __builtin_amdgcn_logf(L) : -INFINITY;
        asm volatile("" : "+v"(inv), "+v"(lam));  // (beside the matrix instructions)
    }
    // ---- publish ----
    if (n16 < G) {
#pragma unroll
        for (int t = 0; t < DT; ++t) {
            const f32x4 x = EXACT ? o[t][0] + o[t][1] : (o[t][0] + o[t][1]) * inv;
            const int off = ((c_rec * G + n16) * kPairRows + (w * DT + t) * 8 + 2 * c4) * 16;
            const u32x4 r0 = {__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(lam), tag};
            const u32x4 r1 = {__float_as_uint(x[2]), __float_as_uint(x[3]), __float_as_uint(lam), tag};
            __builtin_amdgcn_raw_buffer_store_b128(r0, rsrc, off, 0, kAgentScopeAux);
            __builtin_amdgcn_raw_buffer_store_b128(r1, rsrc, off + 16, 0, kAgentScopeAux);
        }
        if (EXACT && w == 0 && c4 == 0) {
            const u32x4 r = {__float_as_uint(L), 0u, __float_as_uint(lam), tag};
            __builtin_amdgcn_raw_buffer_store_b128(r, rsrc, PairLane<G, EXACT>::sum_row(n16, c_rec), 0, kAgentScopeAux);
        }
    }
    // ---- merge (see attn_split_kernel: the same protocol, a bit per unit) ----
    int32_t* counter = counters + bg * kCounterStride;
    unsigned long long* pend = reinterpret_cast<unsigned long long*>(counter + 2);
    uint16_t* out = out_all + bg * G * kD;
    asm volatile("s_barrier" ::: "memory");                                // every wavefront has issued its rows
    if (w == 0) {
        int ticket = 0;
        if (lane == 0) ticket = __hip_atomic_fetch_add(counter, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        ticket = __builtin_amdgcn_readfirstlane(ticket);
        if (ticket == nchunks - 1 && lane == 0) {
            __hip_atomic_store(counter, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);           // next call
            __hip_atomic_store(&epochs[bg], tag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            wait_stores_acknowledged();                                                           // the call number is out before the bits are collected
            sPend = __hip_atomic_exchange(pend, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        if (lane == 0) sTicket = ticket;
    }
    for (int unit = unit0; unit < units; unit += NW * nchunks) {
        if (unit != unit0) at0 = PairLane<G, EXACT>(unit, shift, nchunks);
        if (merge_pairs<G, EXACT>(out, rsrc, at0, nchunks, tag, spin, false)) continue;
        const unsigned long long bit = 1ull << unit;
        uint32_t seen = 0;
        if (lane == 0) {
            const unsigned long long before = __hip_atomic_fetch_or(pend, bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            asm volatile("s_waitcnt vmcnt(0)" :: "v"(before) : "memory");       // the bit is set before the call number is read
            seen = __hip_atomic_load(&epochs[bg], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        seen = __builtin_amdgcn_readfirstlane(seen);
        if (seen == tag) {
            merge_pairs<G, EXACT>(out, rsrc, at0, nchunks, tag, kTagSpinLimit, true);
            if (lane == 0) __hip_atomic_fetch_and(pend, ~bit, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    __syncthreads();
    if (sTicket != nchunks - 1) return false;
    unsigned long long left = sPend;
    for (int k = 0; left != 0; ++k) {
        const int unit = __builtin_ctzll(left);
        left &= left - 1;
        if ((k & (NW - 1)) == w && unit < units) merge_pairs<G, EXACT>(out, rsrc, PairLane<G, EXACT>(unit, shift, nchunks), nchunks, tag, kTagSpinLimit, true);
    }
    return false;
}

// TileParams and the preloaded arguments of a launch.
struct TileArgs { TileParams t; uint32_t rows_heads; int64_t s_b_and_tail; };
static inline TileArgs tile_args(const AttnParams& p) {
    const uint32_t spec_rows = (uint32_t)(p.n_sel < p.cap1 ? p.n_sel : p.cap1);
    TileArgs a{{(float)((double)p.scale * 1.4426950408889634), p.n_sel, p.evict, p.max_rows2, p.cap1, p.cap2, p.slice_spin, p.pred_val,
             p.epochs, p.out, p.counters, p.tag_rows, p.k2, p.v2, p.s2_b, p.s2_h,
             p.pred, p.trig_q_ref, {p.trig_sim}, {p.trig_need}, p.trig_threshold},
            spec_rows | (p.pred != nullptr ? kPredBit : 0) | ((uint32_t)p.Hkv << 16), p.s1_b | (int64_t)((uint64_t)(p.nch | (p.tail_inside ? kTailInside : 0)) << 56)};
    if (p.mark_tail != nullptr) { a.t.mark_tail = p.mark_tail; a.t.mark_count = p.mark_count; }
    return a;
}

}  // namespace rk
