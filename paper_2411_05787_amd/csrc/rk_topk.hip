// rk_topk_select for gfx950: group max + max-pool, then an exact, tie-correct top-K.
//
// The order is decided on the order-preserving 32-bit image of the pooled score P (integer
// compares only, so the result is exact): larger image first, equal images by lower position.
//
// Kernel 1, whole chip (pool_hist_kernel; tiles of 512 positions, of 1024 from 98304 positions on):
//   P[j] = max over the G heads of the group and over the pooling window, staged through LDS so
//   that every weight is read once; P is stored and its top 11 image bits are histogrammed (LDS,
//   then one global atomic per non-empty bin).
// Kernel 2 (select_kernel), workgroups of 1024 threads: from the histogram, the bin b1 that holds
//   the K-th largest score; every position in that bin or a higher one is a candidate (the K
//   winners plus the rest of one bin).  What is listed and ranked are runs of candidates: up to
//   four neighbours with the same pooled score (the pooling window makes neighbours equal, so runs
//   are several times fewer than positions).  Up to 8 workgroups share a row, by rank (select_part):
//   each lists and ranks the runs of its own stretch of scores.  A few long rows are listed by a workgroup per 4096 positions
//   and ranked by the last to arrive (select_listed_kernel, select_listed_batched_kernel).  Up to 256 runs are compared each with
//   each; more, or those of a whole row, are taken into registers and bucket-sorted back into LDS on the
//   64-bit item (P image, position, length): 2048 buckets from the lowest candidate image up to
//   the bin of the 64-th largest score (of equal width, or laid out from the histogram), one more
//   bucket for everything above (fewer than 64 positions); a scan turns bucket counts into
//   offsets, and the rank of a run's first position is the number of positions in the buckets
//   above plus those of the larger runs in its own bucket (a few compares).  Positions that rank
//   below K' are written out directly: idx comes out in rank order.  The kernel also clears the
//   histogram for the next call.
// Dense or degenerate score distributions take further exact steps in kernel 2 (select_row, one workgroup):
// more runs than fit in LDS -> bin b1 is cut once more by the next 11 image bits (one more pass
// over P) and only its upper part stays a candidate; a bucket with more than 1024 runs -> the list
// is bitonic-sorted instead of ranked; still too many candidates (e.g. all scores equal) -> a last
// radix pass (10 bits) finds the K-th largest image T exactly, positions with P > T and the first
// positions with P == T are collected in position order, then bitonic-sorted.
#include "rk_internal.h"
#include "rk_device.h"

namespace rk {

constexpr int kSelThreads = 1024;
constexpr int kSelHeld = 8;                              // vectors of four positions of a row in a thread's registers at a time
constexpr int kBuckets = 2048;                           // regular buckets, plus one for all above
constexpr int kBucketLimit = 1024;                       // larger buckets: sort instead of ranking
constexpr int kAdaptiveFrom = 8192;                      // candidates from which buckets follow the histogram
constexpr int kTopLoose = 64;                            // scores above the bucketed range: fewer than this
constexpr int kPairs = 256;                               // a part's runs up to here are compared each with each
static_assert(kMaxCandidates / 2 * 4 <= 0xFFFF, "buckets of a part count positions in 16 bits");
constexpr int kNonFinite = 1;                            // thread whose two bins of the histogram start at infinity
constexpr int kFineFrom = 4;                             // a bin of more than this many times K' positions is looked at more closely
constexpr int kFineLeast = 1024;                         // ... and of more than this (with few ranks four times K is soon passed, and the look is worth less than it
                                                         // costs: 300 shapes with K from 1 to 300: 0.955 of the time without this bound, one row of 25488, K = 1: 15.4 -> 11.4 us)
constexpr int kPartWords = 8;                            // what a part knows of its stretch
constexpr int kListTile = 4 * kSelThreads;               // positions that a workgroup of select_listed_kernel lists
// Of more candidates than positions fit, more runs than this, or than a 32nd of the row, rank faster in parts (one row of 65537, K = 4096, 6231 runs: 25.3 us, in parts 19.7;
// the longer the row, the more it costs the parts to read: of 262145, K = 10922, 0.9 of the parts' time).
constexpr int kListRuns = 4096;
constexpr int kListTry = 4;                              // runs are listed for up to this many times cand_cap positions
static_assert(kHistBins == 1 << 11, "first-level histogram is 11 bits wide");
static_assert(kHistBins == 2 * kSelThreads, "the selection scans the histogram two bins per thread");
static_assert(((uint32_t)(2 * (kSelThreads - 1 - kNonFinite)) << kHistShift) == 0xFF800000u, "image of infinity");

// What is ranked is a run: up to kRunMax positions next to each other with the same pooled score
// (the pooling window makes the scores of up to pool_w neighbours equal, so there are several
// times fewer runs than candidate positions, and the ranking costs the square of a bucket's
// size).  A run is one 64-bit item: score image | kPosTop - first position | length - 1; larger
// items come first in the selection (two runs never share a first position, so the length never
// decides), and the positions of a run follow each other in the output.
constexpr int kRunMax = 4;                               // a run lies inside one 16-byte vector of scores
constexpr uint32_t kPosTop = (1u << 28) - 1u;            // positions are below RK_MAX_SELECT_LEN = 2^28
static_assert(RK_MAX_SELECT_LEN == (int64_t)kPosTop + 1, "28 bits of an item hold the position");
__device__ __forceinline__ uint64_t item_of(uint32_t key, int j, int len = 1) {
    return ((uint64_t)key << 32) | (uint64_t)(((kPosTop - (uint32_t)j) << 4) | (uint32_t)(len - 1));
}
__device__ __forceinline__ int item_pos(uint64_t item) { return (int)(kPosTop - ((uint32_t)item >> 4)); }
__device__ __forceinline__ uint32_t item_len(uint64_t item) { return ((uint32_t)item & 15u) + 1u; }

template <int TILE>
__global__ __launch_bounds__(256)
void pool_hist_kernel(const float* __restrict__ weights, int64_t w_stride, const int32_t* seq_lens,
                      int32_t max_len, int32_t Hq, int32_t Hkv, int32_t G, int32_t half, int32_t agg,
                      float* __restrict__ pooled, int64_t pooled_stride, uint32_t* __restrict__ hist,
                      const int32_t* pred, int32_t pred_val) {
    const int g = blockIdx.y, b = blockIdx.z;
    if (pred != nullptr && pred[b] != pred_val) return;
    const int len = min(seq_lens[b], max_len);
    const int j0 = blockIdx.x * TILE;
    if (j0 >= len) return;
    __shared__ __attribute__((aligned(16))) float sA[TILE + RK_MAX_POOL_W + 1];
    __shared__ __attribute__((aligned(8))) uint32_t sH[kHistBins];
    const float* wg = weights + ((int64_t)b * Hq + (int64_t)g * G) * w_stride;
    const int span = TILE + 2 * half;
    constexpr int R = (TILE + RK_MAX_POOL_W - 1 + 255) / 256;
    // The heads' weights of every round, all requested together: a head's row is a buffer, what lies outside [0, len) reads as zero (a branch per load made the
    // compiler wait for one before the next).  us per call of rk_topk_select, a round at a time behind branches / as it is, 32 heads over 8: 16 rows of 32768
    // 33.4 / 28.7, 4 of 131072 34.2 / 31.6, 16 of 131072 96.8 / 76.7, one 24.2 / 23.5.  Ahead of the length they gained nothing (24.3), and all of it was lost where
    // max_len is a bound far above it: 65536 of 1048576: 34.6 / 18.2.
    float w[R][RK_MAX_GROUP];
#pragma unroll
    for (int gi = 0; gi < RK_MAX_GROUP; ++gi) {
        if (gi >= G) break;
        const __amdgpu_buffer_rsrc_t row = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(wg + (int64_t)gi * w_stride), 0, len * 4, 0x00020000);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int i = r * 256 + threadIdx.x;
            w[r][gi] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(row, i < span ? (j0 - half + i) * 4 : -4, 0, 0));
        }
    }
    for (int i = threadIdx.x; i < kHistBins; i += 256) sH[i] = 0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (r * 256 >= span) break;
        const int i = r * 256 + threadIdx.x, j = j0 - half + i;
        float a = -INFINITY;                     // outside [0, len): never wins a max
        if (i < span && j >= 0 && j < len) {
#pragma unroll
            for (int gi = 0; gi < RK_MAX_GROUP; ++gi)
                if (gi < G) a = aggregate(a, w[r][gi], gi, agg);
            if (agg == RK_AGG_MEAN) a = __fdiv_rn(a, (float)G);
        }
        if (i < span) sA[i] = a;
    }
    __syncthreads();
    const int64_t bg = (int64_t)b * Hkv + g;
    pool_tile<TILE>(sA, half, j0, len, pooled + bg * pooled_stride, sH);
    __syncthreads();
    flush_histogram(sH, hist + bg * kHistBins);
}

// Inclusive prefix sum over the NT threads of the workgroup, in thread order.  `scratch` holds
// NT / 64 words.  Returns the inclusive sum; *total gets the workgroup sum.
template <int NT>
__device__ __forceinline__ uint32_t block_inclusive_scan(uint32_t v, uint32_t* scratch, uint32_t* total) {
    static_assert(NT / 64 == 16, "a row of lanes adds up the wavefronts");
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint32_t x = wave_inclusive_scan(v);
    lds_barrier();                                // scratch may still be read from a previous scan (loads from memory stay in flight)
    if (lane == 63) scratch[w] = x;
    lds_barrier();
    const uint32_t s = row_inclusive_scan(scratch[lane & 15]);
    const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)s, 15);
    const uint32_t base = w != 0 ? (uint32_t)__builtin_amdgcn_readlane((int)s, w - 1) : 0u;
    *total = tot;
    return x + base;
}

// Given a histogram of NB bins (LDS or global) find the bin that holds the kk-th largest entry,
// counting from the top bin down: sOut[0] = that bin, sOut[1] = entries in higher bins.
// All NT threads call; the result is valid after the call (it ends with a barrier).
template <int NT, int NB>
__device__ void find_bin_from_top(const uint32_t* hist, uint32_t kk, uint32_t* sScan, uint32_t* sOut) {
    constexpr int BPT = NB / NT;
    static_assert(BPT >= 1 && BPT * NT == NB, "bins divide evenly over the threads");
    const int rt = NT - 1 - (int)threadIdx.x;       // thread 0 owns the top bins
    uint32_t h[BPT];
    uint32_t local = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) { h[i] = hist[rt * BPT + i]; local += h[i]; }
    uint32_t total;
    const uint32_t incl = block_inclusive_scan<NT>(local, sScan, &total);   // entries in bins >= BPT*rt
    uint32_t above = incl - local;
    if (above < kk && kk <= incl) {
#pragma unroll
        for (int i = BPT - 1; i >= 0; --i) {
            if (above + h[i] >= kk) { sOut[0] = (uint32_t)(rt * BPT + i); sOut[1] = above; break; }
            above += h[i];
        }
    }
    __syncthreads();
}

// One histogram pass of the slow-path radix select.  On entry the keys still in play are those
// with (key & mask) == prefix and the kk-th largest of them is wanted.  Bins are BITS wide at
// `shift`.  Result in sOut as for find_bin_from_top.
template <int BITS>
__device__ void radix_pass(const float* __restrict__ P, int n, uint32_t prefix, uint32_t mask, int shift,
                           uint32_t kk, uint32_t* sHist, uint32_t* sScan, uint32_t* sOut) {
    constexpr int NB = 1 << BITS;
    const int tid = threadIdx.x;
    for (int i = tid; i < NB; i += kSelThreads) sHist[i] = 0;
    __syncthreads();
    // 16-byte loads, eight of them in flight per thread (rows start 16-byte aligned and are padded
    // to a multiple of four scores); few keys match the prefix, so the atomics are sparse
    const float4* P4 = reinterpret_cast<const float4*>(P);
    const int nvec = (n + 3) >> 2;
    auto count = [&](float v, int j) {
        const uint32_t key = key_of(v);
        if (j < n && (key & mask) == prefix) atomicAdd(&sHist[(key >> shift) & (NB - 1)], 1u);
    };
    constexpr int UN = 8;
    for (int v0 = 0; v0 < nvec; v0 += kSelThreads * UN) {
        float4 pv[UN];
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int v = v0 + u * kSelThreads + tid;
            pv[u] = v < nvec ? P4[v] : make_float4(0.f, 0.f, 0.f, 0.f);
        }
#pragma unroll
        for (int u = 0; u < UN; ++u) {
            const int v = v0 + u * kSelThreads + tid;
            const int j = v < nvec ? v << 2 : n;
            count(pv[u].x, j); count(pv[u].y, j + 1); count(pv[u].z, j + 2); count(pv[u].w, j + 3);
        }
    }
    __syncthreads();
    find_bin_from_top<kSelThreads, NB>(sHist, kk, sScan, sOut);
}

// Sorts sKeys[0 .. npad) descending (npad a power of two); all kSelThreads threads call.
// Wavefront w owns the compare-exchange pairs [w * PW, (w + 1) * PW), PW = npad / 2 / 16.  For a
// stride <= PW those pairs only touch the wavefront's own 2 * PW elements, so such stages are
// separated by a wavefront-local ordering of LDS traffic; only the strides above PW (10 of the
// 78 stages at npad = 4096) need a workgroup barrier.
__device__ void bitonic_sort_desc(uint64_t* sKeys, int npad) {
    constexpr int NWV = kSelThreads / 64;
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int half = npad >> 1;
    if (half < kSelThreads) {
        // small lists: one pair per thread at most, plain barriers
        for (int size = 2; size <= npad; size <<= 1) {
            for (int stride = size >> 1; stride > 0; stride >>= 1) {
                if (tid < half) {
                    const int lo = ((tid & ~(stride - 1)) << 1) | (tid & (stride - 1));
                    const int hi = lo + stride;
                    const bool desc = (lo & size) == 0;
                    const uint64_t a = sKeys[lo], c = sKeys[hi];
                    if ((a < c) == desc) { sKeys[lo] = c; sKeys[hi] = a; }
                }
                __syncthreads();
            }
        }
        return;
    }
    const int PW = half / NWV;                    // pairs per wavefront, a multiple of 64
    bool need_barrier = false;                    // the previous stage crossed wavefront blocks
    for (int size = 2; size <= npad; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            const bool cross = stride > PW;
            if (cross || need_barrier) __syncthreads(); else wave_lds_sync();
            for (int i = w * PW + lane; i < (w + 1) * PW; i += 64) {
                const int lo = ((i & ~(stride - 1)) << 1) | (i & (stride - 1));
                const int hi = lo + stride;
                const bool desc = (lo & size) == 0;
                const uint64_t a = sKeys[lo], c = sKeys[hi];
                if ((a < c) == desc) { sKeys[lo] = c; sKeys[hi] = a; }
            }
            need_barrier = cross;
        }
    }
    __syncthreads();
}

// One (sequence, KV head)'s row, and the workgroup's LDS.
struct SelectRow {
    const float* P;                         // pooled scores, 16-byte aligned
    uint32_t* gh;                           // their first-level histogram
    int n, k, kprime;                       // positions, ranks asked for, ranks that exist
    int room;                               // vectors of four positions that rows have room for
    int cand_cap;
    int32_t* idx; float* sel_scores;        // [k]; sel_scores may be NULL

    __device__ __forceinline__ uint32_t list_limit() const { return (uint32_t)min(kListTry * cand_cap, 0xFFFF); }
    // Vector v of the row as it lies in memory: a buffer, so that nothing branches around a load; behind `room` zeros.
    __device__ __forceinline__ float4 raw4(int v) const {
        const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(P), 0, room * 16, 0x00020000);
        return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, v * 16, 0, 0));
    }
    // ... with positions at and beyond n as -1: below every candidate threshold (scores are >= 0).
    __device__ __forceinline__ float4 load4(int v) const {
        float4 x = raw4(v);
        x.x = 4 * v < n ? x.x : -1.f; x.y = 4 * v + 1 < n ? x.y : -1.f;
        x.z = 4 * v + 2 < n ? x.z : -1.f; x.w = 4 * v + 3 < n ? x.w : -1.f;
        return x;
    }
    // The positions of a run whose first one has rank r, as far as they rank below K'.
    __device__ __forceinline__ void write_run(uint64_t item, uint32_t r) const {
        const int j = item_pos(item);
        const uint32_t len = min(item_len(item), (uint32_t)kprime - min(r, (uint32_t)kprime));
        for (uint32_t i = 0; i < len; ++i) {
            idx[r + i] = j + (int)i;
            if (sel_scores) sel_scores[r + i] = value_of((uint32_t)(item >> 32));
        }
    }
    __device__ __forceinline__ void fill_rest() const {     // ranks that no position has
        for (int i = kprime + (int)threadIdx.x; i < k; i += kSelThreads) {
            idx[i] = -1;
            if (sel_scores) sel_scores[i] = 0.f;
        }
    }
};
struct SelectLds {
    uint64_t* keys;                         // [cand_cap]
    uint32_t* hist;                         // [2 * (kBuckets + 1)]: bucket arrays, or the radix histogram
    uint32_t* scan;                         // [kSelThreads / 64]
    uint32_t* out;                          // [4]
    uint32_t* count;                        // [1]
    uint32_t* part;                         // [kPartWords]
    uint16_t* tab;                          // [kHistBins] buckets of each first-level bin (allocated only if cand_cap > kAdaptiveFrom)

    __device__ __forceinline__ SelectLds(unsigned char* smem, int cand_cap) {
        keys = reinterpret_cast<uint64_t*>(smem);
        hist = reinterpret_cast<uint32_t*>(keys + cand_cap);
        scan = hist + 2 * (kBuckets + 1);
        out = scan + kSelThreads / 64;
        count = out + 4;
        part = count + 1;
        tab = reinterpret_cast<uint16_t*>(part + kPartWords);
    }
};

// Ranks the n_items runs in the list (keys) by buckets and writes them out, the first position after `base` others; hist is cleared.
// False: some bucket holds too many; the list is as it was.
// The list is taken into registers, up to kItems items per thread, so that the same LDS array can receive them again
// sorted by bucket.  A bucket is counted twice in one word, runs << 16 | positions (neither field overflows:
// at most cand_cap runs and 65535 positions in all).
template <class Bucket>
__device__ __forceinline__ bool rank_by_buckets(const SelectRow& row, const SelectLds& lds, uint32_t n_items, uint32_t base, Bucket&& bucket_of) {
    const int tid = threadIdx.x;
    uint64_t* const sKeys = lds.keys;
    uint32_t *const sHist = lds.hist, *const sScan = lds.scan;
    uint32_t* sCnt = sHist;                         // [kBuckets + 1] bucket sizes, then fill marks (in runs)
    uint32_t* sStart = sHist + kBuckets + 1;        // [kBuckets + 1] bucket offsets: runs << 16 | positions
    static_assert(kMaxCandidates < (1 << 16), "runs and positions of a bucket are counted in 16 bits each");
    constexpr int kItems = kMaxCandidates / kSelThreads;
    uint64_t it[kItems];
#pragma unroll
    for (int u = 0; u < kItems; ++u) {
        const int e = u * kSelThreads + tid;
        it[u] = (e < (int)n_items) ? sKeys[e] : 0ull;
    }
    const int n_mine = ((int)n_items - tid + kSelThreads - 1) / kSelThreads;   // items of this thread
    __syncthreads();                                // the list is in registers: sKeys is free
#pragma unroll
    for (int u = 0; u < kItems; ++u)
        if (u < n_mine) atomicAdd(&sCnt[bucket_of((uint32_t)(it[u] >> 32))], 0x10000u | item_len(it[u]));
    __syncthreads();
    // offsets from the top bucket down: thread 0 owns the two highest regular buckets
    const int rt = kSelThreads - 1 - tid;
    const uint32_t c0 = sCnt[2 * rt], c1 = sCnt[2 * rt + 1], cov = sCnt[kBuckets];
    const bool big = (c0 >> 16) > (uint32_t)kBucketLimit || (c1 >> 16) > (uint32_t)kBucketLimit ||
                     (cov >> 16) > (uint32_t)kBucketLimit;
    uint32_t total;
    const uint32_t incl = block_inclusive_scan<kSelThreads>(c0 + c1, sScan, &total);
    const uint32_t above2 = incl - (c0 + c1) + cov;
    if (!__syncthreads_or(big ? 1 : 0)) {
        sStart[2 * rt + 1] = above2;      sCnt[2 * rt + 1] = above2 >> 16;
        sStart[2 * rt] = above2 + c1;     sCnt[2 * rt] = (above2 + c1) >> 16;
        if (tid == 0) { sStart[kBuckets] = 0; sCnt[kBuckets] = 0; }
        __syncthreads();
        // every item into its bucket (order inside a bucket is arbitrary)
#pragma unroll
        for (int u = 0; u < kItems; ++u)
            if (u < n_mine) sKeys[atomicAdd(&sCnt[bucket_of((uint32_t)(it[u] >> 32))], 1u)] = it[u];
        __syncthreads();
        // rank of a run's first position = positions in the buckets above + positions of the
        // larger runs in its own bucket; ranks below K' are the answer
        for (int e = tid; e < (int)n_items; e += kSelThreads) {
            const uint64_t item = sKeys[e];
            const uint32_t bk = bucket_of((uint32_t)(item >> 32));
            const uint32_t st = sStart[bk], lo = st >> 16, hi = sCnt[bk];
            uint32_t r = base + (st & 0xFFFFu);
            // four reads in flight; a read past the bucket's end takes the item itself, which counts nothing
            for (uint32_t x = lo; x < hi; x += 4) {
                uint64_t o[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) o[i] = sKeys[x + i < hi ? x + i : (uint32_t)e];
#pragma unroll
                for (int i = 0; i < 4; ++i) r += (o[i] > item) ? item_len(o[i]) : 0u;
            }
            row.write_run(item, r);
        }
        return true;
    }
    // a huge bucket (many equal or nearly equal scores): put the list back and sort it instead
#pragma unroll
    for (int u = 0; u < kItems; ++u)
        if (u < n_mine) sKeys[u * kSelThreads + tid] = it[u];
    __syncthreads();
    return false;
}

// Sorts the list's nvalid runs and writes them out, the first position after `base` others.
__device__ __forceinline__ void rank_by_sorting(const SelectRow& row, const SelectLds& lds, int nvalid, uint32_t base) {
    const int tid = threadIdx.x;
    uint64_t* const sKeys = lds.keys;
    uint32_t* const sScan = lds.scan;
    int npad = 1;
    while (npad < nvalid) npad <<= 1;
    for (int i = nvalid + tid; i < npad; i += kSelThreads) sKeys[i] = 0;   // sorts behind every real item
    __syncthreads();
    bitonic_sort_desc(sKeys, npad);
    // sKeys[0 .. nvalid) in order: a run's rank is the number of positions in the runs before it.
    // Every thread takes a stretch of the list: the lengths of the stretches before it, then its own.
    {
        const int per = (nvalid + kSelThreads - 1) / kSelThreads;
        const int e0 = min(tid * per, nvalid), e1 = min(e0 + per, nvalid);
        uint32_t mine = 0, total;
        for (int e = e0; e < e1; ++e) mine += item_len(sKeys[e]);
        uint32_t r = block_inclusive_scan<kSelThreads>(mine, sScan, &total) - mine + base;
        for (int e = e0; e < e1; ++e) {
            const uint64_t item = sKeys[e];
            row.write_run(item, r);
            r += item_len(item);
        }
    }
}

// Part number `part` of the selection of one row.
//
// One workgroup alone spends its time on the phases of the ranking (a barrier and some dozen instructions per item and phase, 16
// wavefronts on one CU), so they are shared out by rank: every workgroup reads the whole row and its histogram, cuts the range of
// the candidates' scores into stretches of about the same count (bins of the histogram, cut linearly inside), and lists
// and ranks the runs of its own stretch.  Where its ranks start follows from the histogram and the scores it counts between its
// stretch and the next bin.  Nothing is handed over: the workgroups meet only in the ticket whose last drawer clears the
// histogram, and does the row alone should a stretch not have fitted some workgroup's list (many equal scores).  Where the
// histogram says it (K-th score zero or negative, infinities), the first part does the row, and does not wait for the others.
// What is left to do for this workgroup:
enum SelectLeft { kRowDone, kRowAnew, kRowKnown };       // nothing; the row; the row, with what the histogram says in place (it is cleared by another)
// The ticket: parts that have drawn, those of them that the row does not fit (four bits each), workgroups without a part (select_listed_body).
constexpr uint32_t kDrawn = 1, kDrawnBad = 0x10, kDrawnIdle = 0x100;
__device__ __forceinline__ uint32_t draw_ticket(int32_t* ticket, uint32_t what) {
    return (uint32_t)__hip_atomic_fetch_add(ticket, (int32_t)what, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// All threads of a workgroup, with what has been drawn, its own included: the last one leaves the workspace clean, or has the row to do.
__device__ __forceinline__ SelectLeft after_drawing(const SelectRow& row, int32_t* ticket, uint32_t drawn, int lg_parts, int idle) {
    if ((drawn & ~(kDrawnIdle - kDrawnBad)) != (1u << lg_parts) + (uint32_t)idle * kDrawnIdle) return kRowDone;
    if (threadIdx.x == 0) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if ((drawn & (kDrawnIdle - kDrawnBad)) != 0) {           // (the ranks that others have written come out the same)
        __syncthreads();
        return kRowAnew;
    }
    row.gh[2 * threadIdx.x] = 0; row.gh[2 * threadIdx.x + 1] = 0;
    return kRowDone;
}
// What bounds it is latency: us after the first workgroup's first instruction, 8 rows of 32768 positions, K = 2048, medians:
// lengths 0.7, histogram and stretch 2.6, row looked through 3.8, runs listed 5.5, ranked 6.7, written 7.1 (the launch 9 - 10
// against 10.6 before); of 131072, K = 8192, 32 parts: 0.8, 2.7, 6.6, 10.5 (512 KB through one CU), 11.9, 12.4.
__device__ __forceinline__ SelectLeft select_part(const SelectRow& row, const SelectLds& lds, int32_t* __restrict__ ticket, const int part, const int lg_parts,
                                                  const int idle, uint2& h01) {
    const int tid = threadIdx.x, n = row.n, kprime = row.kprime, nvec = (n + 3) >> 2, cand_cap = row.cand_cap;
    uint64_t* const sKeys = lds.keys;
    uint32_t *const sHist = lds.hist, *const sScan = lds.scan, *const sOut = lds.out, *const sCount = lds.count, *const sPart = lds.part;
    const int list_cap = cand_cap / 2;      // runs a part lists; the other half of the room is the queue's
    uint32_t* const sQueue = reinterpret_cast<uint32_t*>(sKeys + list_cap);                // [cand_cap]
    uint32_t* const gh = row.gh;
    // This thread's two bins of the first-level histogram are requested first, the row's scores (whatever its length: rows have room
    // for max_len) behind them: the bins are counted while the scores are on their way.
    const int rt = kSelThreads - 1 - tid;
    h01 = *reinterpret_cast<const uint2*>(gh + 2 * rt);
    constexpr int NV = kSelHeld;
    float4 held[NV];
#pragma unroll
    for (int u = 0; u < NV; ++u) held[u] = row.raw4(u * kSelThreads + tid);

    // The stretch is [B(part + 1), B(part)): B(i) leaves i / parts of the K' ranks above it, the last one all candidates.  sPart: this
    // part's B(i), the end of B(i)'s bin, the positions above that bin; B(i + 1); positions with an infinite score or NaN; vectors
    // queued; positions between the stretch and the end of the bin; positions in the stretch.  sOut: as in select_row.
    if (tid == 0) { *sCount = 0; sPart[5] = 0; sPart[6] = 0; sPart[7] = 0; }
    for (int i = tid; i < kBuckets + 1; i += kSelThreads) sHist[i] = 0;
    const uint32_t h0 = h01.x, h1 = h01.y;
    const uint32_t t0 = ((uint32_t)kprime * (uint32_t)part) >> lg_parts, t1 = ((uint32_t)kprime * (uint32_t)(part + 1)) >> lg_parts;
    {
        uint32_t total;
        const uint32_t incl = block_inclusive_scan<kSelThreads>(h0 + h1, sScan, &total);   // entries in bins >= 2 rt
        const uint32_t abv = incl - (h0 + h1);
        const uint32_t kk1 = (uint32_t)kprime, kk2 = min((uint32_t)kprime, (uint32_t)kTopLoose);
        if (abv < kk1 && kk1 <= incl) {
            const bool upper = abv + h1 >= kk1;
            sOut[0] = (uint32_t)(2 * rt + (upper ? 1 : 0));
            sOut[1] = upper ? abv : abv + h1;
            sOut[2] = upper ? h1 : h0;
        }
        if (abv < kk2 && kk2 <= incl) sOut[3] = (uint32_t)(2 * rt + (abv + h1 >= kk2 ? 1 : 0));
        {                                       // (stretches in bits of scores >= 0)
            if (tid == kNonFinite) sPart[4] = incl;
            const uint32_t spare = part + 1 == 1 << lg_parts ? last_spare(kk1) : 0u;
            // (the bin above thread 64 i's upper one is another wavefront's: no ratio there)
            const uint32_t h2 = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)h0, 0x138, 0xF, 0xF, true);      // wave_shr:1
            auto bound = [&](uint32_t t, uint32_t spare) {
                const bool upper = abv + h1 >= t;
                const uint32_t bin = (uint32_t)(2 * rt + (upper ? 1 : 0)), h = upper ? h1 : h0;
                return stretch_bound(t, spare, ((bin + 1u) << kHistShift) - 0x80000000u, 1u << kHistShift, upper ? abv : abv + h1, h,
                                     density_ratio(bin, h, upper ? h2 : h1));
            };
            if (t0 == 0) {                  // (the top, or fewer ranks than parts)
                if (tid == 0) { sPart[0] = sPart[1] = 0x80000000u; sPart[2] = 0; }
            } else if (abv < t0 && t0 <= incl) {
                const StretchBound b = bound(t0, 0u);
                sPart[0] = b.at; sPart[1] = b.end; sPart[2] = b.above;
            }
            if (t1 == 0) {
                if (tid == 0) sPart[3] = 0x80000000u;
            } else if (abv < t1 && t1 <= incl) {
                sPart[3] = bound(t1, spare).at;
            }
        }
        lds_barrier();
    }
    // the lowest and highest candidates' bits (scores as whole numbers)
    if (sOut[0] <= (uint32_t)kHistBins / 2 || sPart[4] != 0) {      // the same in every part
        lds_barrier();
        if (tid == 0) sPart[4] = draw_ticket(ticket, kDrawn) + kDrawn;
        __syncthreads();
        after_drawing(row, ticket, sPart[4], lg_parts, idle);        // (nobody's row is bad here)
        return part == 0 ? kRowKnown : kRowDone;
    }
    const uint32_t b1 = sOut[0], above1 = sOut[1], in1 = sOut[2], key_top = (sOut[3] + 1u) << kHistShift;
    // The K'-th score lies anywhere in its bin, and that bin may hold many times the ranks that are left: the last part starts
    // with an estimate of its lower end and takes the rest of the bin only if too few positions turn up.  (131072 positions with half of
    // the keys near 64 centroids, K = 8192: 4136 runs in the last part without it, 350 in the others; a step of one layer 105.8 ->
    // 101.3 us.  The second look at the row costs 4 - 8 us: with 3/16 of the ranks to spare instead of 3/8 that step takes 110, a window
    // of 32 queries over 32768 positions 70.9 instead of 67.7.)
    const bool last = part + 1 == 1 << lg_parts;
    bool hopeless = false;
    uint32_t hi = sPart[0], end = sPart[1], above_end = sPart[2], estimate = sPart[3], floor = last ? (b1 << kHistShift) - 0x80000000u : estimate;
    if (in1 > max((uint32_t)(kprime * kFineFrom), (uint32_t)kFineLeast) && t1 > above1) {
        // The K'-th score's bin (no other can) holds many times the ranks there are, which says little about where in it they lie:
        // one look at the row counts its scores by the next 11 bits (a dozen LDS atomics per thread and 32768 positions at the least:
        // from twice K positions on instead of four times it cost votes of 20 queries over 131072 rows 11 us of 109).  Scores that differ
        // little, 8 rows, us per call: one workgroup or spread-out listing / parts without this look, bins taken as even / now: e^(0.05 N(0, 1)),
        // 8000 positions, K = 500: 22.3 / 28.3 / 14.7, 131072, K = 8192: 83 / 115 / 36; e^(0.25 N(0, 1)), pooled by 7, where the densities of the
        // bins do: 14.0 / 16.7 / 12.0 and 33.0 / 37.1 / 25.2.  (Equal scores throughout, 8 rows of 2000: 29.3 / 31.8 / 34.5, of 32768 100 / 101 / 104.)
        constexpr int kSub = kHistShift - 11;
        const uint32_t from = (b1 << kHistShift) - 0x80000000u;
        for (int v0 = 0; v0 < nvec; v0 += NV * kSelThreads) {
            float4 next[NV];
#pragma unroll
            for (int u = 0; u < NV; ++u) next[u] = row.raw4(v0 + (NV + u) * kSelThreads + tid);
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                if (v0 + u * kSelThreads >= nvec) break;
                const int in = n - ((v0 + u * kSelThreads + tid) << 2);         // positions of the vector inside the row
                const uint32_t none = 0xBF800000u;
                const uint32_t a = in > 0 ? __float_as_uint(held[u].x) : none, b = in > 1 ? __float_as_uint(held[u].y) : none;
                const uint32_t c = in > 2 ? __float_as_uint(held[u].z) : none, d = in > 3 ? __float_as_uint(held[u].w) : none;
                const int ed = d == c ? 1 : 0, ec = c == b ? 1 + ed : 0, eb = b == a ? 1 + ec : 0;
                auto count = [&](uint32_t bits, int len) {
                    if (bits - from < 1u << kHistShift) atomicAdd(&sHist[(bits - from) >> kSub], (uint32_t)len);
                };
                count(a, 1 + eb);
                if (b != a) count(b, 1 + ec);
                if (c != b) count(c, 1 + ed);
                if (d != c) count(d, 1);
            }
#pragma unroll
            for (int u = 0; u < NV; ++u) held[u] = next[u];
        }
        // (so many in a 2^-13th of an octave are equal scores: some part's list would not do)
        auto closer = [&](uint32_t t, uint32_t spare) {
            find_bin_from_top<kSelThreads, 1 << 11>(sHist, t - above1, sScan, sOut);
            const uint32_t sub = sOut[0], over = sOut[1], h = sHist[sub];
            hopeless = hopeless || h > (uint32_t)cand_cap;
            return stretch_bound(t, spare, from + ((sub + 1u) << kSub), 1u << kSub, above1 + over, h, 1.f);
        };
        lds_barrier();
        if (t0 > above1) {
            const StretchBound b = closer(t0, 0u);
            hi = b.at; end = b.end; above_end = b.above;
        }
        const StretchBound b = closer(t1, last ? last_spare((uint32_t)kprime) : 0u);
        estimate = b.at;
        floor = last ? b.end - (b.above == t1 ? 0u : 1u << kSub) : estimate;       // (above all ranks: the whole of its bin)
        lds_barrier();
        for (int i = tid; i < kBuckets + 1; i += kSelThreads) sHist[i] = 0;
#pragma unroll
        for (int u = 0; u < NV; ++u) held[u] = row.raw4(u * kSelThreads + tid);
    }
    // (few positions in the bin are taken whole: 9 rows of 37290, K = 19: 20.0 -> 16.0 us, without the second look)
    uint32_t lo = last && in1 <= (uint32_t)kPairs ? floor : stretch_low(estimate, floor, hi);
    uint32_t top = hi, top_end = end;       // the stretch so far, and what is looked for in this pass over the row
    while (lo < top && !hopeless) {
        // Bits of scores as whole numbers, from the stretch's lowest.  A vector of four positions with none in the stretch or
        // between it and the end of its bin is passed over after one comparison of the least; the numbers of the others are
        // queued, so that what is left to do with them takes every lane.
        const uint32_t stretch = top - lo, upto = top_end - lo, more = upto - stretch;
        for (int v0 = 0; v0 < nvec; v0 += NV * kSelThreads) {
            float4 next[NV];
#pragma unroll
            for (int u = 0; u < NV; ++u) next[u] = row.raw4(v0 + (NV + u) * kSelThreads + tid);
            uint64_t hit[NV];
            int found = 0;
            const int left = nvec - v0 - tid;           // (what lies behind the row is whatever the workspace holds)
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const uint32_t ra = __float_as_uint(held[u].x) - lo, rb = __float_as_uint(held[u].y) - lo;
                const uint32_t rc = __float_as_uint(held[u].z) - lo, rd = __float_as_uint(held[u].w) - lo;
                hit[u] = __ballot(min(min(ra, rb), min(rc, rd)) < upto && u * kSelThreads < left);
                found += __popcll(hit[u]);
            }
            if (found != 0) {
                int at = 0;
                if ((tid & 63) == 0) at = (int)atomicAdd(&sPart[5], (uint32_t)found);
                at = __builtin_amdgcn_readfirstlane(at);
#pragma unroll
                for (int u = 0; u < NV; ++u) {
                    const int q = at + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(hit[u] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)hit[u], 0u));
                    if ((hit[u] >> (tid & 63) & 1) != 0 && q < cand_cap) sQueue[q] = (uint32_t)(v0 + u * kSelThreads + tid);
                    at += __popcll(hit[u]);
                }
            }
#pragma unroll
            for (int u = 0; u < NV; ++u) held[u] = next[u];
        }
        lds_barrier();
        const int queued = min((int)sPart[5], cand_cap);
        uint32_t higher = 0, inside = 0;
        for (int e0 = 0; e0 < queued; e0 += kSelThreads) {
            const int e = e0 + tid;
            if (e - (tid & 63) >= queued) break;        // (whole wavefronts)
            uint32_t a = 0xBF800000u, b = a, c = a, d = a;
            int j = 0;
            if (e < queued) {
                const int v = (int)sQueue[e];
                const float4 x = row.raw4(v);
                j = v << 2;
                const int in = n - j;                   // positions of the vector inside the row
                a = __float_as_uint(x.x);
                b = in > 1 ? __float_as_uint(x.y) : b; c = in > 2 ? __float_as_uint(x.z) : c; d = in > 3 ? __float_as_uint(x.w) : d;
            }
            const uint32_t ra = a - lo, rb = b - lo, rc = c - lo, rd = d - lo;
            higher += (ra - stretch < more ? 1u : 0u) + (rb - stretch < more ? 1u : 0u) + (rc - stretch < more ? 1u : 0u) +
                      (rd - stretch < more ? 1u : 0u);
            inside += (ra < stretch ? 1u : 0u) + (rb < stretch ? 1u : 0u) + (rc < stretch ? 1u : 0u) + (rd < stretch ? 1u : 0u);
            // the runs (up to four neighbours with the same score) among them
            const bool fa = ra < stretch, fb = rb < stretch && b != a, fc = rc < stretch && c != b, fd = rd < stretch && d != c;
            const uint32_t runs = (fa ? 1u : 0u) + (fb ? 1u : 0u) + (fc ? 1u : 0u) + (fd ? 1u : 0u);
            const uint32_t incl = wave_inclusive_scan(runs);
            uint32_t at = 0;
            if ((tid & 63) == 63) at = atomicAdd(sCount, incl);
            uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)at, 63) + incl - runs;
            auto put = [&](uint32_t bits, int first, int len) {
                if (pos < (uint32_t)list_cap) sKeys[pos] = item_of(bits | 0x80000000u, first, len);      // runs beyond the end are only counted
                ++pos;
            };
            const int ed = d == c ? 1 : 0, ec = c == b ? 1 + ed : 0, eb = b == a ? 1 + ec : 0;
            if (fa) put(a, j, 1 + eb);
            if (fb) put(b, j + 1, 1 + ec);
            if (fc) put(c, j + 2, 1 + ed);
            if (fd) put(d, j + 3, 1);
        }
        if (top_end != top) {
            higher = wave_inclusive_scan(higher);
            if ((tid & 63) == 63 && higher != 0) atomicAdd(&sPart[6], higher);
        }
        if (lo == floor) break;
        inside = wave_inclusive_scan(inside);
        if ((tid & 63) == 63 && inside != 0) atomicAdd(&sPart[7], inside);
        lds_barrier();
        if (above_end + sPart[6] + sPart[7] >= (uint32_t)kprime) break;
        if (sPart[5] > (uint32_t)cand_cap) break;       // (the queue was too short: what was counted is not all)
        top = top_end = lo;
        lo = floor;
        lds_barrier();
        if (tid == 0) sPart[5] = 0;
        lds_barrier();
#pragma unroll
        for (int u = 0; u < NV; ++u) held[u] = row.raw4(u * kSelThreads + tid);
    }
    lds_barrier();
    const uint32_t n_items = *sCount, base = above_end + sPart[6];
    const bool bad = hopeless || sPart[5] > (uint32_t)cand_cap || n_items > (uint32_t)list_cap;
    const uint32_t mine = bad ? kDrawn + kDrawnBad : kDrawn;
    uint32_t seen = 0;                      // (every thread has read the histogram; the answer is waited for behind the ranking)
    if (tid == 0) seen = draw_ticket(ticket, mine);
    if (!bad && n_items != 0) {
        if (n_items <= (uint32_t)kPairs) {
            // few runs: every one against every other, a wavefront for 64 of them and a share of the others
            const int w = __builtin_amdgcn_readfirstlane(tid >> 6), lg = n_items > 64 ? n_items > 128 ? 2 : 1 : 0;
            const int shares = kSelThreads / 64 >> lg, share = w >> lg, e = (w & ((1 << lg) - 1)) * 64 + (tid & 63);
            {
                const uint64_t item = e < (int)n_items ? sKeys[e] : ~0ull;
                uint32_t r = 0;
#pragma unroll 4
                for (int x = share; x < (int)n_items; x += shares) {
                    const uint64_t o = sKeys[x];
                    r += o > item ? item_len(o) : 0u;
                }
                if (r != 0) atomicAdd(&sHist[e], r);
            }
            lds_barrier();                  // (leaves the ticket on its way)
            if (tid < (int)n_items) row.write_run(sKeys[tid], base + sHist[tid]);
        } else {
            // equal widths; the first part's thin top in one bucket (see select_row)
            const uint32_t from = lo + 0x80000000u, to = part == 0 && key_top > from ? key_top : hi + 0x80000000u;
            const uint32_t width = to - 1u - from;
            const int shift = width >= (uint32_t)kBuckets ? 32 - 11 - __builtin_clz(width) : 0;
            if (!rank_by_buckets(row, lds, n_items, base, [&](uint32_t key) { return min((key - from) >> shift, (uint32_t)kBuckets); }))
                rank_by_sorting(row, lds, (int)n_items, base);
        }
    }
    if (part == 0) row.fill_rest();
    if (tid == 0) sOut[0] = seen + mine;
    __syncthreads();
    return after_drawing(row, ticket, sOut[0], lg_parts, idle);
}

// From the histogram, in one scan from the top bin down (thread 0 owns the top two bins):
// the bin b1 that holds the K'-th largest score (with the count above it), and the bin that
// holds the kTopLoose-th largest, which bounds the bucketed range from above so that the one
// bucket for "everything above" stays small (its items are ranked by a loop over the bucket).
__device__ __forceinline__ void scan_histogram(const SelectRow& row, const SelectLds& lds, uint2 h01) {
    const int tid = threadIdx.x, rt = kSelThreads - 1 - tid;
    const uint32_t h0 = h01.x, h1 = h01.y;
    if (tid == 0) *lds.count = 0;
    for (int i = tid; i < kBuckets + 1; i += kSelThreads) lds.hist[i] = 0;     // bucket sizes of the fast path
    uint32_t total;
    const uint32_t incl = block_inclusive_scan<kSelThreads>(h0 + h1, lds.scan, &total);   // entries in bins >= 2 rt
    const uint32_t abv = incl - (h0 + h1);
    const uint32_t kk1 = (uint32_t)row.kprime, kk2 = min((uint32_t)row.kprime, (uint32_t)kTopLoose);
    if (abv < kk1 && kk1 <= incl) {
        const bool upper = abv + h1 >= kk1;
        lds.out[0] = (uint32_t)(2 * rt + (upper ? 1 : 0));
        lds.out[1] = upper ? abv : abv + h1;
        lds.out[2] = upper ? h1 : h0;
    }
    if (abv < kk2 && kk2 <= incl) lds.out[3] = (uint32_t)(2 * rt + (abv + h1 >= kk2 ? 1 : 0));
}

// The runs of candidates inside one vector of four scores (positions j .. j + 3; a candidate is
// a score >= thr; scores are >= +0 and -0 never occurs, so equal scores have equal bits and the
// order-preserving image is the bit pattern with the top bit set): count_runs() counts them,
// visit_runs() calls visit(image, first position, length) for each, in position order.
__device__ __forceinline__ uint32_t count_runs(const float4 x, float thr) {
    const uint32_t a = __float_as_uint(x.x), b = __float_as_uint(x.y), c = __float_as_uint(x.z), d = __float_as_uint(x.w);
    return (x.x >= thr ? 1u : 0u) + (x.y >= thr && b != a ? 1u : 0u) + (x.z >= thr && c != b ? 1u : 0u) +
           (x.w >= thr && d != c ? 1u : 0u);
}
template <class Visit>
__device__ __forceinline__ void visit_runs(const float4 x, int j, float thr, Visit&& visit) {
    const uint32_t a = __float_as_uint(x.x), b = __float_as_uint(x.y), c = __float_as_uint(x.z), d = __float_as_uint(x.w);
    const int ed = d == c ? 1 : 0;                       // positions after j + 2 with its score
    const int ec = c == b ? 1 + ed : 0;                  // ... after j + 1
    const int eb = b == a ? 1 + ec : 0;                  // ... after j
    if (x.x >= thr) visit(a | 0x80000000u, j, 1 + eb);
    if (x.y >= thr && b != a) visit(b | 0x80000000u, j + 1, 1 + ec);
    if (x.z >= thr && c != b) visit(c | 0x80000000u, j + 2, 1 + ed);
    if (x.w >= thr && d != c) visit(d | 0x80000000u, j + 3, 1);
}
static_assert(kRunMax == 4, "runs are found inside one float4");

constexpr int kNotListed = -1;              // instead of the number of a row's candidate runs that lds.keys holds already

// The whole selection of one row by one workgroup.  known: h01 and lds.out are what the histogram says of it, and LDS is as below after the scan.
template <bool ADAPT>                    // ADAPT: compiled with the histogram-driven bucket layout (large K only)
__device__ __forceinline__ void select_row(const SelectRow& row, const SelectLds& lds, uint2 h01, const bool known, const int listed) {
    const int tid = threadIdx.x, n = row.n, kprime = row.kprime, nvec = (n + 3) >> 2, cand_cap = row.cand_cap;
    uint64_t* const sKeys = lds.keys;
    uint32_t *const sHist = lds.hist, *const sScan = lds.scan, *const sOut = lds.out, *const sCount = lds.count;
    uint16_t* const sTab = lds.tab;
    const float* const P = row.P;
    uint32_t* const gh = row.gh;
    // The first 32 scores of every thread (the whole row up to 32768 positions) are requested now, behind this thread's two bins of
    // the histogram, 16-byte loads all in flight together, and stay in registers.
    const int rt = kSelThreads - 1 - tid;
    if (!known) h01 = *reinterpret_cast<const uint2*>(gh + 2 * rt);
    constexpr int NV = kSelHeld;
    float4 held[NV];
    if (listed < 0) {
#pragma unroll
        for (int u = 0; u < NV; ++u) held[u] = row.load4(u * kSelThreads + tid);
    }

    const uint32_t h0 = h01.x, h1 = h01.y;
    if (!known) {
        scan_histogram(row, lds, h01);
        gh[2 * rt] = 0; gh[2 * rt + 1] = 0;                     // cleared for the next call
        __syncthreads();
    }
    const uint32_t b1 = sOut[0];
    const uint32_t above = sOut[1];
    uint32_t count_ge = above + sOut[2];
    const uint32_t key_top = (sOut[3] + 1u) << kHistShift;      // sOut[3] >= b1; wraps to 0 for the last bin

    uint32_t key_thr = b1 << kHistShift;
    // The list holds runs, so it may have room where the positions are too many: up to
    // kListTry * cand_cap positions the runs are listed anyway, counted as they are, and the list
    // is used if they fit.  (Bucket offsets below are counted in 16 bits: 65535 positions at most.)
    const bool try_list = count_ge <= row.list_limit();

    uint32_t n_items = 0;                   // runs in the list
    float thr = value_of(key_thr);                       // lowest candidate score (scores are >= 0)
    // The runs of candidates among NV vectors per thread (vector u of the thread is number
    // v0 + u * kSelThreads + tid of the row) go to the end of the list in sKeys: every wavefront
    // counts its own, reserves the room with one LDS atomic and writes them there.  The order of
    // the list depends on the order of the reservations; nothing after it depends on that order.
    auto list_candidates = [&](const float4 (&x)[NV], int v0) {
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < NV; ++u) c += count_runs(x[u], thr);
        const uint32_t incl = wave_inclusive_scan(c);
        const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (tot == 0) return;                                      // the same in all 64 lanes
        uint32_t base = 0;
        if ((tid & 63) == 63) base = atomicAdd(sCount, tot);
        uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)base, 63) + incl - c;
#pragma unroll
        for (int u = 0; u < NV; ++u)
            visit_runs(x[u], (v0 + u * kSelThreads + tid) << 2, thr, [&](uint32_t key, int j, int len) {
                if (pos < (uint32_t)cand_cap) sKeys[pos] = item_of(key, j, len);    // runs beyond the end are only counted
                ++pos;
            });
    };
    // One pass over the row, which is the only work here that is proportional to n: the vectors
    // held in registers first, the rest of a longer row NV vectors per thread at a time, all of
    // them in flight together.  Returns the number of runs (they are in sKeys if they fit).
    bool held_is_row_start = true;
    auto list_row = [&]() -> uint32_t {
        if (!held_is_row_start) {
#pragma unroll
            for (int u = 0; u < NV; ++u) held[u] = row.load4(u * kSelThreads + tid);
        }
        list_candidates(held, 0);
        for (int v0 = NV * kSelThreads; v0 < nvec; v0 += kSelThreads * NV) {
#pragma unroll
            for (int u = 0; u < NV; ++u) held[u] = row.load4(v0 + u * kSelThreads + tid);
            list_candidates(held, v0);
            held_is_row_start = false;
        }
        __syncthreads();
        const uint32_t runs = *sCount;
        __syncthreads();
        if (tid == 0) *sCount = 0;
        return runs;
    };
    // Candidates are the positions whose image is >= key_thr.  Normally that is "bin b1 or above"; if their runs are too many for
    // LDS, bin b1 is cut once more by the next 11 image bits.
    uint32_t prefix = key_thr, mask = 0x7FFu << kHistShift, kk = (uint32_t)kprime - above;   // radix-select state
    bool refined = false;
    bool in_lds = false;                    // the runs of all candidates are in sKeys
    if (listed >= 0) {
        n_items = (uint32_t)listed;
        in_lds = true;
    } else if (try_list) {
        n_items = list_row();
        in_lds = n_items <= (uint32_t)cand_cap;
    }
    if (!in_lds) {                          // (more than cand_cap positions: fewer would have been listed)
        radix_pass<11>(P, n, prefix, mask, 10, kk, sHist, sScan, sOut);
        const uint32_t b2 = sOut[0];
        count_ge = above + sOut[1] + sHist[b2];
        prefix |= b2 << 10; mask |= 0x7FFu << 10; kk -= sOut[1];
        key_thr = prefix;
        thr = value_of(key_thr);
        refined = true;
        __syncthreads();
        if (count_ge <= (uint32_t)cand_cap) {
            n_items = list_row();
            in_lds = true;
        }
    }
    // bucket width: the smallest power of two for which [key_thr, key_top) fits in kBuckets buckets
    const uint32_t span = key_top - 1u - key_thr;        // 11 significant bits are left after the shift
    const int bucket_shift = span >= (uint32_t)kBuckets ? 32 - 11 - __builtin_clz(span) : 0;

    // Buckets of the fast path.  Preferred layout: every first-level bin from b1 up to the bin of
    // the kTopLoose-th largest score gets a power-of-two number of equal-width buckets in
    // proportion to its count in the histogram, so that all buckets hold about the same number of
    // candidates however the scores are distributed over the octaves (scores thin out towards the
    // top: equal-width buckets over the whole range leave most candidates in the lowest few, and
    // the ranking below costs the square of a bucket's size).  sTab[bin] = first bucket | log2 of
    // the number of buckets << 11.  Used from kAdaptiveFrom candidates on (below that, building the
    // table costs more than it saves: measured).  Otherwise, and when the threshold is not on a bin
    // boundary or the bins need more than kBuckets buckets: equal-width buckets over the whole range.
    bool adaptive = false;
    auto bucket_of = [&](uint32_t key) -> uint32_t {
        if (ADAPT && adaptive) {
            if (key_top != 0u && key >= key_top) return (uint32_t)kBuckets;
            const uint32_t t = sTab[key >> kHistShift], e = t >> 11;
            return (t & 0x7FFu) + ((key >> (kHistShift - e)) & ((1u << e) - 1u));
        }
        return min((key - key_thr) >> bucket_shift, (uint32_t)kBuckets);
    };
    int nvalid;                             // entries of sKeys that are real (sorting paths)
    if (in_lds) {
        // ---- candidates = every position whose image is >= key_thr, count_ge of them; their runs are in LDS ----
        if (refined) {                                  // the radix pass used the array: clear it again
            for (int i = tid; i < kBuckets + 1; i += kSelThreads) sHist[i] = 0;
        }
        if (ADAPT && !refined && count_ge > (uint32_t)kAdaptiveFrom) {
            const uint32_t top = (key_top - 1u) >> kHistShift;
            const float per_item = 1400.f / (float)count_ge;              // aims at ~1500 buckets in all
            auto log2_buckets = [&](uint32_t h, uint32_t bin) -> int {    // -1: no bucket
                if (h == 0 || bin < b1 || bin > top) return -1;
                const float x = (float)h * per_item;
                return x <= 1.f ? 0 : min((int)(__log2f(x) + 0.5f), 11);
            };
            const int e0 = log2_buckets(h0, 2 * rt), e1 = log2_buckets(h1, 2 * rt + 1);
            const uint32_t nb0 = e0 < 0 ? 0u : 1u << e0, nb1 = e1 < 0 ? 0u : 1u << e1;
            uint32_t total;
            const uint32_t incl = block_inclusive_scan<kSelThreads>(nb0 + nb1, sScan, &total);   // buckets of bins >= 2 rt
            adaptive = total != 0 && total <= (uint32_t)kBuckets;
            if (adaptive) {
                const uint32_t first0 = total - incl;                     // buckets of all lower bins
                if (e0 >= 0) sTab[2 * rt] = (uint16_t)(first0 | ((uint32_t)e0 << 11));
                if (e1 >= 0) sTab[2 * rt + 1] = (uint16_t)((first0 + nb0) | ((uint32_t)e1 << 11));
            }
            __syncthreads();
        }
        if (rank_by_buckets(row, lds, n_items, 0u, bucket_of)) {
            row.fill_rest();
            return;
        }
        nvalid = (int)n_items;
    } else {
        // ---- slow path: exact K-th largest image T by radix select over P ----
        // (bin b1 has been cut by the next 11 image bits above: 10 bits are left)
        __syncthreads();
        radix_pass<10>(P, n, prefix, mask, 0, kk, sHist, sScan, sOut);
        const uint32_t T = prefix | sOut[0];
        const uint32_t need_eq = kk - sOut[1];          // >= 1 positions with image == T are taken
        const uint32_t n_gt = (uint32_t)kprime - need_eq;
        __syncthreads();
        uint32_t base_eq = 0;
        for (int tile0 = 0; tile0 < n; tile0 += kSelThreads) {
            const int j = tile0 + tid;
            const bool in = j < n;
            const uint32_t key = in ? key_of(P[j]) : 0u;
            if (in && key > T) sKeys[atomicAdd(sCount, 1u)] = item_of(key, j);
            const bool eq = in && key == T;
            if (base_eq < need_eq) {                    // uniform over the workgroup
                if (__syncthreads_or(eq ? 1 : 0)) {
                    uint32_t total;
                    const uint32_t incl = block_inclusive_scan<kSelThreads>(eq ? 1u : 0u, sScan, &total);
                    const uint32_t rank = base_eq + incl - 1u;
                    if (eq && rank < need_eq) sKeys[n_gt + rank] = item_of(key, j);
                    base_eq += total;
                }
            }
        }
        nvalid = kprime;                                // runs of one position each
    }
    rank_by_sorting(row, lds, nvalid, 0u);
    row.fill_rest();
}

template <bool ADAPT>
__device__ __forceinline__
void select_body(const float* __restrict__ pooled, int64_t pooled_stride, const int32_t* seq_lens,
                 int32_t max_len, int32_t k, uint32_t* __restrict__ hist, int32_t cand_cap,
                 int32_t* __restrict__ idx, float* __restrict__ sel_scores,
                 const int32_t* pred, int32_t pred_val,
                 int32_t* __restrict__ sel_counters, const int b, const int g, const int Hkv,
                 const int part, const int lg_parts) {
    if (pred != nullptr && pred[b] != pred_val) return;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const SelectLds lds(smem, cand_cap);
    const int64_t bg = (int64_t)b * Hkv + g;
    const int n = min(seq_lens[b], max_len);
    const SelectRow row{pooled + bg * pooled_stride, hist + bg * kHistBins, n, k, min(k, max(n, 0)), (max_len + 3) >> 2, cand_cap, idx + bg * k,
                        sel_scores ? sel_scores + bg * k : nullptr};
    if (row.kprime <= 0) {                  // nothing was histogrammed for an empty sequence
        if (part == 0) row.fill_rest();
        return;
    }
    uint2 h01 = make_uint2(0, 0);
    const SelectLeft left = lg_parts > 0 ? select_part(row, lds, sel_counters + bg * 2, part, lg_parts, 0, h01) : kRowAnew;
    if (left != kRowDone) select_row<ADAPT>(row, lds, h01, left == kRowKnown, kNotListed);
}

// A row among a few long ones (select_listed): this workgroup's 4096 positions; the last to arrive ranks.  Where the candidates hardly
// fit one list (scores that crowd in the K-th one's bin), the first workgroups take the row by parts instead: the last to
// arrive would have to look through all of it by itself, several times (4 rows of 262145, K = 10922, scores in clusters: 2.5 times the parts' time).
template <bool ADAPT>
__device__ __forceinline__
void select_listed_body(const float* __restrict__ pooled, int64_t pooled_stride, const int32_t* seq_lens,
                        int32_t max_len, int32_t k, uint32_t* __restrict__ hist, int32_t cand_cap,
                        int32_t* __restrict__ idx, float* __restrict__ sel_scores,
                        const int32_t* pred, int32_t pred_val,
                        int32_t* __restrict__ sel_counters, uint64_t* __restrict__ cand_list, const int b, const int g, const int Hkv) {
    if (pred != nullptr && pred[b] != pred_val) return;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const SelectLds lds(smem, cand_cap);
    const int tid = threadIdx.x, tile = blockIdx.x;
    const int64_t bg = (int64_t)b * Hkv + g;
    const int n = min(seq_lens[b], max_len);
    const SelectRow row{pooled + bg * pooled_stride, hist + bg * kHistBins, n, k, min(k, max(n, 0)), (max_len + 3) >> 2, cand_cap, idx + bg * k,
                        sel_scores ? sel_scores + bg * k : nullptr};
    if (row.kprime <= 0) {                  // nothing was histogrammed for an empty sequence
        if (tile == 0) row.fill_rest();
        return;
    }
    const int rt = kSelThreads - 1 - tid;
    uint2 h01 = *reinterpret_cast<const uint2*>(row.gh + 2 * rt);
    const float4 x = row.load4(tile * kSelThreads + tid), sample = row.load4(tid);
    scan_histogram(row, lds, h01);
    __syncthreads();
    const float thr = value_of(lds.out[0] << kHistShift);
    const uint32_t candidates = lds.out[1] + lds.out[2];
    bool list_it = candidates <= (uint32_t)cand_cap;           // (all of this the same in every workgroup of the row)
    if (!list_it && candidates <= row.list_limit()) {          // their runs, going by the row's first positions
        const uint32_t some = (sample.x >= thr ? 1u : 0u) + (sample.y >= thr ? 1u : 0u) + (sample.z >= thr ? 1u : 0u) + (sample.w >= thr ? 1u : 0u);
        uint32_t total;
        (void)block_inclusive_scan<kSelThreads>(count_runs(sample, thr) << 16 | some, lds.scan, &total);
        list_it = total != 0 && candidates * (total >> 16) <= (total & 0xFFFFu) * (uint32_t)min(cand_cap - cand_cap / 8, max(kListRuns, n >> 5));
    }
    SelectLeft left = kRowKnown;
    int runs = kNotListed;
    if (!list_it || lds.out[0] < (uint32_t)kHistBins / 2) {
        constexpr int kLgParts = 3, kParts = 1 << kLgParts;
        static_assert((kListFrom + kListTile - 1) / kListTile >= kParts && kListRows * kParts <= kComputeUnits, "a listed row has workgroups for its parts");
        const int idle = (int)gridDim.x - kParts;
        int32_t* ticket = sel_counters + bg * 2;
        if (tile < kParts) {
            left = select_part(row, lds, ticket, tile, kLgParts, idle, h01);
        } else {
            if (tid == 0) lds.part[0] = draw_ticket(ticket, kDrawnIdle) + kDrawnIdle;
            __syncthreads();
            left = after_drawing(row, ticket, lds.part[0], kLgParts, idle);
        }
        if (left == kRowDone) return;
    } else {
        int32_t* n_listed = sel_counters + bg * 2;
        int32_t* arrived = n_listed + 1;
        uint64_t* list = cand_list + bg * cand_cap;
        const uint32_t c = count_runs(x, thr);
        uint32_t total;
        const uint32_t incl = block_inclusive_scan<kSelThreads>(c, lds.scan, &total);
        if (tid == 0 && total != 0)
            *lds.count = (uint32_t)__hip_atomic_fetch_add(n_listed, (int32_t)total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        uint32_t pos = *lds.count + incl - c;
        visit_runs(x, (tile * kSelThreads + tid) << 2, thr, [&](uint32_t key, int j, int len) {
            if (pos < (uint32_t)cand_cap)                      // runs beyond the list's end are only counted
                __hip_atomic_store(&list[pos], item_of(key, j, len), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            ++pos;
        });
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");       // the list entries are acknowledged
        __syncthreads();                                       // ... and every thread has read the histogram
        if (tid == 0) lds.part[0] = (uint32_t)__hip_atomic_fetch_add(arrived, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
        if (lds.part[0] != gridDim.x - 1) return;
        // last to arrive: everything of this row is in (a workgroup has the answer of its reservation before it writes its
        // entries, hence before its ticket: the count is final); leave the workspace clean, then rank
        if (tid == 0) {
            lds.part[1] = (uint32_t)__hip_atomic_load(n_listed, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(n_listed, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __hip_atomic_store(arrived, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            *lds.count = 0;
        }
        row.gh[2 * rt] = 0; row.gh[2 * rt + 1] = 0;
        __syncthreads();
        if (lds.part[1] <= (uint32_t)cand_cap) runs = (int)lds.part[1];
        for (int e = tid; e < runs; e += kSelThreads) lds.keys[e] = __hip_atomic_load(&list[e], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __syncthreads();
    }
    select_row<ADAPT>(row, lds, h01, left == kRowKnown, runs);
}

// Grid (workgroups of a row, KV heads, sequences).
template <bool ADAPT>
__global__ __launch_bounds__(kSelThreads)
void select_listed_kernel(const float* __restrict__ pooled, int64_t pooled_stride, const int32_t* seq_lens,
                          int32_t max_len, int32_t k, uint32_t* __restrict__ hist, int32_t cand_cap,
                          int32_t* __restrict__ idx, float* __restrict__ sel_scores,
                          const int32_t* pred, int32_t pred_val, int32_t* __restrict__ sel_counters, uint64_t* __restrict__ cand_list) {
    select_listed_body<ADAPT>(pooled, pooled_stride, seq_lens, max_len, k, hist, cand_cap, idx, sel_scores, pred, pred_val,
                              sel_counters, cand_list, (int)blockIdx.z, (int)blockIdx.y, (int)gridDim.y);
}

// Grid (KV heads, parts, sequences): consecutive workgroups go to the 8 XCDs in turn, so with 8 KV heads (or 4, or 16) the parts of
// a row share an L2.
template <bool ADAPT>
__global__ __launch_bounds__(kSelThreads)
void select_kernel(const float* __restrict__ pooled, int64_t pooled_stride, const int32_t* seq_lens,
                   int32_t max_len, int32_t k, uint32_t* __restrict__ hist, int32_t cand_cap,
                   int32_t* __restrict__ idx, float* __restrict__ sel_scores,
                   const int32_t* pred, int32_t pred_val, int32_t* __restrict__ sel_counters) {
    select_body<ADAPT>(pooled, pooled_stride, seq_lens, max_len, k, hist, cand_cap, idx, sel_scores, pred, pred_val,
                       sel_counters, (int)blockIdx.z, (int)blockIdx.x, (int)gridDim.x, (int)blockIdx.y, 31 - __builtin_clz(gridDim.y));
}

// The selections of several layers in one launch: grid z = layer * batch + sequence; what differs
// from layer to layer comes from a table passed by value.
struct SelectBatch {
    const float* pooled[kBatchLayers];
    uint32_t* hist[kBatchLayers];
    int32_t* idx[kBatchLayers];
    int32_t* sel_counters[kBatchLayers];
    const int32_t* pred[kBatchLayers];       // NULL: every sequence of the layer
};

template <bool ADAPT>
__global__ __launch_bounds__(kSelThreads)
void select_batched_kernel(const SelectBatch tab, int32_t batch, int64_t pooled_stride, const int32_t* seq_lens,
                           int32_t max_len, int32_t k, int32_t cand_cap, int32_t pred_val) {
    const int layer = blockIdx.z / batch, b = blockIdx.z - layer * batch;
    select_body<ADAPT>(tab.pooled[layer], pooled_stride, seq_lens, max_len, k, tab.hist[layer], cand_cap, tab.idx[layer],
                       nullptr, tab.pred[layer], pred_val, tab.sel_counters[layer], b, (int)blockIdx.x, (int)gridDim.x,
                       (int)blockIdx.y, 31 - __builtin_clz(gridDim.y));
}

// ... of a few long rows in all layers together: grid (workgroups of a row, KV heads, layer * batch + sequence).
struct ListBatch {
    SelectBatch rows;
    uint64_t* cand_list[kListRows];
};

template <bool ADAPT>
__global__ __launch_bounds__(kSelThreads)
void select_listed_batched_kernel(const ListBatch tab, int32_t batch, int64_t pooled_stride, const int32_t* seq_lens,
                                  int32_t max_len, int32_t k, int32_t cand_cap, int32_t pred_val) {
    const int layer = blockIdx.z / batch, b = blockIdx.z - layer * batch;
    select_listed_body<ADAPT>(tab.rows.pooled[layer], pooled_stride, seq_lens, max_len, k, tab.rows.hist[layer], cand_cap, tab.rows.idx[layer],
                              nullptr, tab.rows.pred[layer], pred_val, tab.rows.sel_counters[layer], tab.cand_list[layer], b,
                              (int)blockIdx.y, (int)gridDim.y);
}

}  // namespace rk

using namespace rk;

namespace rk {

int pool_stage(const rk_geom* geom, const float* weights, int64_t w_stride, const int32_t* seq_lens,
               int32_t max_len, int32_t pool_w, int32_t agg, const int32_t* pred, int32_t pred_val,
               const Workspace& ws, hipStream_t st) {
    const int G = geom->n_q_heads / geom->n_kv_heads;
    const int tile = pool_tile_for(max_len);
    dim3 pgrid((max_len + tile - 1) / tile, geom->n_kv_heads, geom->batch);
    if (tile == kPoolTileLong)
        hipLaunchKernelGGL((pool_hist_kernel<kPoolTileLong>), pgrid, dim3(256), 0, st, weights, w_stride, seq_lens, max_len,
                           geom->n_q_heads, geom->n_kv_heads, G, (pool_w - 1) / 2, agg, ws.pooled, pooled_row_stride(max_len), ws.hist,
                           pred, pred_val);
    else
        hipLaunchKernelGGL((pool_hist_kernel<kPoolTile>), pgrid, dim3(256), 0, st, weights, w_stride, seq_lens, max_len,
                           geom->n_q_heads, geom->n_kv_heads, G, (pool_w - 1) / 2, agg, ws.pooled, pooled_row_stride(max_len), ws.hist,
                           pred, pred_val);
    return launch_status();
}

int check_select_args(int32_t k, int32_t pool_w, int32_t agg, int32_t max_len) {
    if (pool_w < 1 || (pool_w & 1) == 0) return RK_ERR_INVALID_ARG;
    if (pool_w > RK_MAX_POOL_W || k > RK_MAX_K || agg < RK_AGG_MAX || agg > RK_AGG_FIRST) return RK_ERR_UNSUPPORTED;
    if ((int64_t)max_len > RK_MAX_SELECT_LEN) return RK_ERR_UNSUPPORTED;
    return RK_OK;
}

template <bool ADAPT>
static int launch_select(const rk_geom* geom, const int32_t* seq_lens, int32_t max_len, int32_t k, int32_t* idx,
                         float* sel_scores, const int32_t* pred, int32_t pred_val, const Workspace& ws, hipStream_t st) {
    // the sort kernel may need more than the default dynamic LDS; the per-bin bucket table is part
    // of it only where there can be kAdaptiveFrom candidates
    const size_t lds = (size_t)ws.cand_cap * sizeof(uint64_t) +
                       (2 * (kBuckets + 1) + kSelThreads / 64 + 4 + 1 + kPartWords) * sizeof(uint32_t) +
                       (ADAPT ? kHistBins * sizeof(uint16_t) : 0);
    const int64_t rows = (int64_t)geom->batch * geom->n_kv_heads;
    const bool listed = ws.cand_list != nullptr && select_listed(max_len, k, rows);
    static size_t lds_allowed = 48 * 1024;       // grows monotonically (one per instantiation)
    if (lds > lds_allowed) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&select_kernel<ADAPT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&select_listed_kernel<ADAPT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
            (void)hipGetLastError();
            return RK_ERR_UNSUPPORTED;
        }
        lds_allowed = lds;
    }
    if (listed) {
        dim3 lgrid((max_len + kListTile - 1) / kListTile, geom->n_kv_heads, geom->batch);
        hipLaunchKernelGGL((select_listed_kernel<ADAPT>), lgrid, dim3(kSelThreads), lds, st, ws.pooled, pooled_row_stride(max_len), seq_lens,
                           max_len, k, ws.hist, ws.cand_cap, idx, sel_scores, pred, pred_val, ws.sel_counters, ws.cand_list);
        return launch_status();
    }
    dim3 sgrid(geom->n_kv_heads, select_parts(rows), geom->batch);
    hipLaunchKernelGGL((select_kernel<ADAPT>), sgrid, dim3(kSelThreads), lds, st, ws.pooled, pooled_row_stride(max_len), seq_lens,
                       max_len, k, ws.hist, ws.cand_cap, idx, sel_scores, pred, pred_val, ws.sel_counters);
    return launch_status();
}

template <bool ADAPT>
static int launch_select_batched(const rk_geom* geom, int n_layers, const Workspace* wss, int32_t* const* idx,
                                 const int32_t* seq_lens, int32_t max_len, int32_t k, const int32_t* const* pred,
                                 int32_t pred_val, hipStream_t st) {
    const int cand_cap = wss[0].cand_cap;
    const size_t lds = (size_t)cand_cap * sizeof(uint64_t) +
                       (2 * (kBuckets + 1) + kSelThreads / 64 + 4 + 1 + kPartWords) * sizeof(uint32_t) +
                       (ADAPT ? kHistBins * sizeof(uint16_t) : 0);
    static size_t lds_allowed = 48 * 1024;
    if (lds > lds_allowed) {
        if (hipFuncSetAttribute(reinterpret_cast<const void*>(&select_batched_kernel<ADAPT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess ||
            hipFuncSetAttribute(reinterpret_cast<const void*>(&select_listed_batched_kernel<ADAPT>),
                                hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds) != hipSuccess) {
            (void)hipGetLastError();
            return RK_ERR_UNSUPPORTED;
        }
        lds_allowed = lds;
    }
    const int64_t problems = (int64_t)(n_layers < kBatchLayers ? n_layers : kBatchLayers) * geom->batch * geom->n_kv_heads;
    const bool listed = wss[0].cand_list != nullptr && select_listed(max_len, k, problems);      // (no more than kListRows layers then)
    const int parts = select_parts(problems);
    for (int l0 = 0; l0 < n_layers; l0 += kBatchLayers) {
        const int n = n_layers - l0 < kBatchLayers ? n_layers - l0 : kBatchLayers;
        SelectBatch tab{};
        for (int l = 0; l < n; ++l) {
            const Workspace& w = wss[l0 + l];
            tab.pooled[l] = w.pooled; tab.hist[l] = w.hist; tab.idx[l] = idx[l0 + l];
            tab.sel_counters[l] = w.sel_counters;
            tab.pred[l] = pred ? pred[l0 + l] : nullptr;
        }
        if (listed) {
            ListBatch list{tab, {}};
            for (int l = 0; l < n; ++l) list.cand_list[l] = wss[l].cand_list;
            dim3 lgrid((max_len + kListTile - 1) / kListTile, geom->n_kv_heads, n * geom->batch);
            hipLaunchKernelGGL((select_listed_batched_kernel<ADAPT>), lgrid, dim3(kSelThreads), lds, st, list, (int32_t)geom->batch,
                               pooled_row_stride(max_len), seq_lens, max_len, k, (int32_t)cand_cap, pred_val);
            return launch_status();
        }
        dim3 grid(geom->n_kv_heads, parts, n * geom->batch);
        hipLaunchKernelGGL((select_batched_kernel<ADAPT>), grid, dim3(kSelThreads), lds, st, tab, (int32_t)geom->batch,
                           pooled_row_stride(max_len), seq_lens, max_len, k, (int32_t)cand_cap, pred_val);
        const int rc = launch_status();
        if (rc != RK_OK) return rc;
    }
    return RK_OK;
}

int select_batched_stage(const rk_geom* geom, int n_layers, const Workspace* wss, int32_t* const* idx,
                         const int32_t* seq_lens, int32_t max_len, int32_t k, const int32_t* const* pred, int32_t pred_val,
                         hipStream_t st) {
    if ((int64_t)kBatchLayers * geom->batch > 65535) return RK_ERR_UNSUPPORTED;      // grid z
    for (int l = 1; l < n_layers; ++l)
        if (wss[l].cand_cap != wss[0].cand_cap) return RK_ERR_INVALID_ARG;
    if (wss[0].cand_cap > kAdaptiveFrom) return launch_select_batched<true>(geom, n_layers, wss, idx, seq_lens, max_len, k, pred, pred_val, st);
    return launch_select_batched<false>(geom, n_layers, wss, idx, seq_lens, max_len, k, pred, pred_val, st);
}

// Two builds of the selection kernel: the one with the histogram-driven bucket layout serves the
// workspaces that can hold more than kAdaptiveFrom candidates (K > 4096); the other is the same
// code without it, because the smaller kernel measures faster where the layout is never used
// (1 us per layer of a full step at K = 2048 when it runs beside the attention kernel).
int select_stage(const rk_geom* geom, const int32_t* seq_lens, int32_t max_len, int32_t k, int32_t* idx,
                 float* sel_scores, const int32_t* pred, int32_t pred_val, const Workspace& ws, hipStream_t st) {
    if (ws.cand_cap > kAdaptiveFrom)
        return launch_select<true>(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, st);
    return launch_select<false>(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, st);
}

}  // namespace rk

extern "C" int rk_topk_select(const rk_geom* geom, const float* weights, int64_t w_stride,
                              const int32_t* seq_lens, int32_t max_len,
                              int32_t k, int32_t pool_w, int32_t agg,
                              int32_t* idx, float* sel_scores,
                              const int32_t* pred, int32_t pred_val,
                              void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!weights || !seq_lens || !idx || max_len <= 0 || k <= 0 || w_stride < max_len) return RK_ERR_INVALID_ARG;
    if ((rc = check_select_args(k, pool_w, agg, max_len)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, k, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    if ((rc = pool_stage(geom, weights, w_stride, seq_lens, max_len, pool_w, agg, pred, pred_val, ws, st)) != RK_OK) return rc;
    return select_stage(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, st);
}

extern "C" int rk_full_attn_select(const rk_geom* geom, const void* q, rk_kv full,
                                   const int32_t* seq_lens, int32_t max_len,
                                   void* out, float* weights, int64_t w_stride, float* lse,
                                   int32_t k, int32_t pool_w, int32_t agg,
                                   int32_t* idx, float* sel_scores,
                                   const int32_t* pred, int32_t pred_val,
                                   void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!q || !out || !seq_lens || !idx || max_len <= 0 || k <= 0) return RK_ERR_INVALID_ARG;
    if (!aligned16(q) || ((uintptr_t)out & 1u)) return RK_ERR_INVALID_ARG;
    if ((rc = check_kv(full)) != RK_OK) return rc;
    if (weights && (w_stride < max_len || ((uintptr_t)weights & 3u))) return RK_ERR_INVALID_ARG;
    if ((rc = check_select_args(k, pool_w, agg, max_len)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, k, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    rc = full_attn_stage(geom, q, full, seq_lens, max_len, out, weights, w_stride, lse, pred, pred_val, ws, st,
                         false, (pool_w - 1) / 2, false, agg);
    if (rc != RK_OK) return rc;
    return select_stage(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, st);
}

extern "C" int rk_score_select(const rk_geom* geom, const void* q, rk_kv full,
                               const int32_t* seq_lens, int32_t max_len,
                               float* weights, int64_t w_stride, float* lse,
                               int32_t k, int32_t pool_w, int32_t agg,
                               int32_t* idx, float* sel_scores,
                               const int32_t* pred, int32_t pred_val,
                               void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!q || !seq_lens || !idx || max_len <= 0 || k <= 0) return RK_ERR_INVALID_ARG;
    if (!aligned16(q)) return RK_ERR_INVALID_ARG;
    if ((rc = check_kv(full, false)) != RK_OK) return rc;
    if (weights && (w_stride < max_len || ((uintptr_t)weights & 3u))) return RK_ERR_INVALID_ARG;
    if ((rc = check_select_args(k, pool_w, agg, max_len)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, k, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    rc = full_attn_stage(geom, q, full, seq_lens, max_len, nullptr, weights, w_stride, lse, pred, pred_val, ws, st,
                         false, (pool_w - 1) / 2, true, agg);
    if (rc != RK_OK) return rc;
    return select_stage(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, st);
}

extern "C" int rk_full_attn_pool(const rk_geom* geom, const void* q, rk_kv full,
                                 const int32_t* seq_lens, int32_t max_len,
                                 void* out, float* weights, int64_t w_stride, float* lse,
                                 int32_t pool_w, int32_t agg, int32_t /*beside_other_work*/,
                                 const int32_t* pred, int32_t pred_val,
                                 void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!q || !out || !seq_lens || max_len <= 0) return RK_ERR_INVALID_ARG;
    if (!aligned16(q) || ((uintptr_t)out & 1u)) return RK_ERR_INVALID_ARG;
    if ((rc = check_kv(full)) != RK_OK) return rc;
    if (weights && (w_stride < max_len || ((uintptr_t)weights & 3u))) return RK_ERR_INVALID_ARG;
    if ((rc = check_select_args(1, pool_w, agg, max_len)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, 0, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    return full_attn_stage(geom, q, full, seq_lens, max_len, out, weights, w_stride, lse, pred, pred_val, ws,
                           (hipStream_t)stream, false, (pool_w - 1) / 2, false, agg);
}

extern "C" int rk_full_attn_deferred(const rk_geom* geom, const void* q, rk_kv full,
                                     const int32_t* seq_lens, int32_t max_len, void* out, float* lse,
                                     const int32_t* pred, int32_t pred_val,
                                     void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!q || !out || !seq_lens || max_len <= 0) return RK_ERR_INVALID_ARG;
    if (!aligned16(q) || ((uintptr_t)out & 1u)) return RK_ERR_INVALID_ARG;
    if ((rc = check_kv(full)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, 0, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    return full_attn_stage(geom, q, full, seq_lens, max_len, out, nullptr, 0, lse, pred, pred_val, ws,
                           (hipStream_t)stream, false, 0, false, RK_AGG_MAX, true);
}

extern "C" int rk_select_pooled(const rk_geom* geom, const int32_t* seq_lens, int32_t max_len, int32_t k,
                                int32_t* idx, float* sel_scores, const int32_t* pred, int32_t pred_val,
                                void* workspace, size_t workspace_bytes, void* stream) {
    int rc = check_geom(geom);
    if (rc != RK_OK) return rc;
    if (!seq_lens || !idx || max_len <= 0 || k <= 0) return RK_ERR_INVALID_ARG;
    if ((rc = check_select_args(k, 1, RK_AGG_MAX, max_len)) != RK_OK) return rc;
    Workspace ws;
    if ((rc = check_workspace(geom, max_len, k, workspace, workspace_bytes, &ws)) != RK_OK) return rc;
    return select_stage(geom, seq_lens, max_len, k, idx, sel_scores, pred, pred_val, ws, (hipStream_t)stream);
}
