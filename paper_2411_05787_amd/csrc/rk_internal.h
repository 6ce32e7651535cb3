// Shared host-side plumbing of the library: workspace layout, argument checks, launch checks.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stddef.h>
#include <math.h>

#include "../../include/refreshkv.h"

namespace rk {

constexpr int kD = RK_HEAD_DIM;          // head_dim
constexpr int kMinChunk = 128;           // rows one workgroup takes per round: 4 wavefronts x 32
constexpr int kMaxChunks = 256;          // most partial results one (sequence, KV head) produces
constexpr int kMergeChunks = 64;         // ... when the split kernel itself merges them
#ifndef RK_TARGET_WGS
#define RK_TARGET_WGS 768                // workgroups a split launch aims for where its caller says nothing else
#endif

// Workgroups per (sequence, KV head) of a split attention launch whose partial results a second
// kernel merges.  Upper bound: as many as give the launch `target` workgroups in all, never more than
// `limit` (the most partial results the merge takes), never more than there are stretches of kMinChunk rows.
// Below that bound, a count that gives every CU the same number of workgroups is preferred
// (total a multiple of the 256 CUs) as long as no wavefront gets more tiles for it.  Measured on
// the score-emitting kernel alone, compiled for three workgroups per CU then (K straight into the operand layout), 8 KV
// heads, total workgroups -> us per launch:
//   24576 rows: 512 -> 20.5, 768 -> 21.5, 1024 -> 22.4;   560..720 -> 22.5..25.9
//   32768 rows: 512 -> 27.1, 768 -> 27.5, 1024 -> 26.6;   560..720 -> 28.9..31.6
//   65536 rows: 512 -> 51.5, 768 -> 52.5, 1024 -> 49.7;   560..720 -> 54.5..60.1
// and the same picture with 4 KV heads and with a batch of 4: an even spread is worth 10-20%,
// which of the even spreads is worth 3-5% and depends on the length (emit_split_target decides there).
constexpr int kComputeUnits = 256;
static inline int split_workgroups(int64_t max_rows, int64_t n_problems, int limit, int target = RK_TARGET_WGS) {
    if (n_problems < 1) n_problems = 1;
    int64_t per = target / n_problems;
    const int64_t stretches = (max_rows + kMinChunk - 1) / kMinChunk;
    if (per > stretches) per = stretches;
    if (per > limit) per = limit;
    if (per < 1) per = 1;
    const int64_t tiles = (max_rows + 31) / 32;
    auto rounds = [&](int64_t nch) { return (tiles + 4 * nch - 1) / (4 * nch); };
    // (a total that is a multiple of kComputeUnits: every unit-th count)
    const int64_t low = n_problems & -n_problems, unit = low < kComputeUnits ? kComputeUnits / low : 1;
    for (int64_t nch = per / unit * unit; nch >= 1 && 8 * nch >= 5 * per; nch -= unit)
        if (rounds(nch) == rounds(per)) return (int)nch;
    return (int)per;
}

// Workgroups per (sequence, KV head) when the last workgroup of the launch merges the partial
// results inside the kernel (partial steps; short full steps without scores).  There the merge
// sets the terms (measured, K = 1024..8192, groups of 4, 7 and 8): it reads the partial outputs
// in batches of 16 per round trip, and a 17th partial result costs 0.8 us, about what a whole
// further round of tiles costs a wavefront (16 workgroups: 9.1 us, 17: 9.9 at K = 2048; 16: 10.3,
// 33: 13.7 at K = 4096; 16: 14.6, 40: 17.2 at K = 8192).  So: the largest count within whole
// batches of 16 that keeps the rounds per wavefront at 5 or fewer, one batch if possible; and a
// tail of a few rows (the tokens decoded since the refresh) gets no workgroup of its own, one
// wavefront takes it as a second tile.  With several sequences the launch as a whole is best at
// about one workgroup per CU (us per launch by workgroups per (sequence, KV head), 8 KV heads:
// 16 sequences, K = 1024: 1: 21.7, 2: 18.7, 4: 19.5, 6: 20.7, 8: 23.4;  16 x 2048: 2: 28.4, 4: 31.1,
// 6: 33.8, 16: 40.0;  8 x 4096: 2: 33.0, 4: 28.5, 12: 32.1, 32: 45.1;  4 x 2048: 4: 16.5, 8: 13.7,
// 16: 14.1;  64 x 512: 1: 30.1, 2: 33.6), so the upper bound is 256 workgroups in all, not the 768 of
// the kernels that leave the merge to a second launch.
// two_batches: the ticketed merge, which requests two batches of 16 partial outputs before it waits
// for the first: 32 partial results cost it one round trip, so where 16 workgroups would leave every
// wavefront two or more tiles, 32 halve the tiles for nothing (one sequence, 4 KV heads, 7 heads per
// group: K = 4096 10.4 -> 10.0 us, K = 8192 13.8 -> 12.5; 48 and 64 workgroups: 10.3 / 13.0 and more; the
// tagged merge reads 20 partial results per round trip and more rows per result: 32 cost it 16.2
// against 13.0 us at K = 8192, groups of 4).
// (Groups of up to 4 heads: the tagged merge wins while 16 workgroups give a wavefront one tile, the
// ticketed one with 32 workgroups beyond: K = 2048 7.5 / 7.7 us, 4096 9.8 / 9.3, 8192 13.0 / 12.5,
// 16384 23.9 / 18.1; so where this is true and the merge is the last workgroup's, the partial step takes the
// ticketed form whatever the group.  With the merge by slices, below, neither is used for launches over few
// pairs: what is left of this rule serves the workspace without a tagged region.)
static inline bool two_batches_pay(int64_t rows, int64_t tail_rows, int64_t n_problems) {
    const int64_t problems = n_problems > 0 ? n_problems : 1;
    const int64_t main_rows = (rows > 0 && tail_rows <= kMinChunk) ? rows : rows + tail_rows;     // a few rows decoded since the refresh do not count
    return (kComputeUnits + problems / 2) / problems >= 32 && (main_rows + 31) / 32 > 4 * 16;
}
static inline int merged_split_workgroups(int64_t rows, int64_t tail_rows, int64_t n_problems, bool two_batches = false) {
    const int64_t all_rows = rows + tail_rows;
    const int64_t counted = (rows > 0 && tail_rows <= 32) ? rows : all_rows;
    const int64_t problems = n_problems > 0 ? n_problems : 1;
    int64_t per = (kComputeUnits + problems / 2) / problems;        // one workgroup per CU in all, see above
    const int64_t stretches = (counted + kMinChunk - 1) / kMinChunk;
    if (per > stretches) per = stretches;
    if (per > kMergeChunks) per = kMergeChunks;
    if (per < 1) per = 1;
    const int64_t tiles = (all_rows + 31) / 32;
    if (two_batches && two_batches_pay(rows, tail_rows, n_problems)) return 32;
    for (int64_t n = 16; n < per; n += 16)
        if ((tiles + 4 * n - 1) / (4 * n) <= 5) return (int)n;
    return (int)per;
}

// The same for the tagged merge (groups of up to 4 heads) from 16 (sequence, KV head) pairs on; first for 32 and more.
// With many pairs the launch is bound by what a CU gets through, not by one workgroup's chain:
// it takes about (workgroups per CU, rounded up) x (tiles per wavefront + 1 for a workgroup's
// fixed costs), plus a round trip of the merge per 20 partial results beyond the first 20.  A
// total just above a multiple of the 256 CUs is what hurts: the few CUs with one workgroup more set
// the time.  `tail` = 1: the rows decoded since the refresh have a workgroup of their own.
// Measured, us per launch, old rule -> this one (8 KV heads, groups of 4): 16 sequences, K = 1024:
// 22.1 -> 18.9; K = 2048: 37.1 -> 32.3; K = 4096: 68.3 -> 54.1; 8 sequences, K = 1024: 14.6 -> 12.8;
// K = 2048: 23.7 -> 20.6; 4 sequences, K = 2048: 14.4 -> 13.0; K = 8192: 38.2 -> 29.9; 32 x 1024:
// 38.3 -> 33.8 - 35.5; 64 x 512: 39.9 -> 35.0.
// With 16 to 31 pairs (2 or 3 sequences of 8 KV heads) the workgroups that share a CU overlap their
// fixed costs, so only the tiles count twice there: (tiles per wavefront + 1) + (workgroups per CU - 1) x
// tiles per wavefront, fewer tiles per wavefront on a tie (3 sequences, K = 2048: 288 workgroups 12.7 -> 408
// workgroups 10.4; K = 4096: 17.5 -> 14.7; K = 8192: 29.7 -> 25.2; 2 sequences, K = 4096: 272 workgroups
// 13.9 -> 192 or 256 workgroups 12.3; K = 8192: 22.1 -> 18.1 - 18.4; K = 2048 stays at 272 workgroups, 9.8).
// The rows decoded since the refresh: a workgroup of their own (*tail_own = 1) or one wavefront's extra tile at the
// end (0), whichever the same estimate likes better; without their workgroups the launch can be exactly one
// workgroup per CU (16 sequences of 8 KV heads: K = 2048, 2 workgroups per pair and no tail workgroup, 256 in all,
// 28.7 us against 3 + 1, 512 in all, 32.6; K = 1024: 17.5 against 18.3; 8 sequences, K = 2048: 4 per pair 19.4
// against 20.0).  tail_rows > 128 (or no selected rows): all rows are shared out alike.
static inline int batched_tagged_workgroups(int64_t rows, int64_t tail_rows, int* tail_own, int64_t n_problems) {
    const bool small_tail = rows > 0 && tail_rows > 0 && tail_rows <= kMinChunk;
    const int64_t main_rows = small_tail ? rows : rows + tail_rows;
    const int64_t stretches = (main_rows + kMinChunk - 1) / kMinChunk;
    const int64_t tiles = (main_rows + 31) / 32;
    const bool few = n_problems < 32;
    int64_t best = 1, best_cost = -1, best_rounds = 0;
    int best_tail = 0;
    for (int tail = small_tail ? 1 : 0; tail >= 0; --tail) {
        for (int64_t n = 1; n <= stretches && n <= kMergeChunks; ++n) {
            const int64_t per_cu = ((n + tail) * n_problems + kComputeUnits - 1) / kComputeUnits;
            const int64_t rounds = (tiles + 4 * n - 1) / (4 * n);
            const int64_t fixed = 1 + (n + tail - 1) / 20;
            const int64_t extra = (small_tail && !tail) ? 1 : 0;          // the tail as one wavefront's last tile
            const int64_t cost = (few ? rounds + fixed + (per_cu - 1) * rounds : per_cu * (rounds + fixed)) + extra;
            if (best_cost < 0 || cost < best_cost || (few && cost == best_cost && tail == best_tail && rounds < best_rounds)) {   // ties (few pairs): fewer tiles per wavefront
                best = n; best_cost = cost; best_rounds = rounds; best_tail = tail;
            }
        }
    }
    *tail_own = best_tail;
    return (int)best;
}

// The same where the partial results are merged by slices (every workgroup its share: see attn_split_kernel) and
// the launch has at most 8 (sequence, KV head) pairs.  That merge costs a workgroup about the same whatever the
// number of partial results (a lane reads a quarter of them), so the tiles per wavefront decide: as many workgroups
// as give every wavefront the fewest tiles, within what the merge takes (`limit` partial results per pair) and what
// is resident at once (two workgroups per compute unit); the fewest workgroups among those.  A few rows decoded
// since the refresh (tail_rows <= 128) do not count: they get a workgroup of their own (*tail_own = 1) unless that
// one more partial result would cost every wavefront a tile; then one wavefront takes them as a second tile
// (K = 8192, one sequence of 8 KV heads: 64 workgroups 11.2 us, 63 + 1: 13.6, the ticketed form with 32: 12.3;
// 4 KV heads of 7 query heads: 10.1 / 10.7 / 12.8).  Measured against the sizing above, us per partial step, one
// sequence: 8 KV heads, K = 3072: 8.8 -> 7.4, 6144: 11.0 -> 10.0, 12288: 17.1 -> 14.9, 16384: 21.5 -> 18.8;
// 4 KV heads of 7: K = 3072: 8.8 -> 7.4, 4096: 9.0 -> 7.7, 6144: 11.2 -> 8.7, 8192: 12.7 -> 10.3.  (With 12 pairs
// it was no gain: 3 sequences of 4 KV heads, K = 8192: 15.3 -> 16.2.)
static inline int sliced_split_workgroups(int64_t rows, int64_t tail_rows, int* tail_own, int64_t n_problems, int limit) {
    const int64_t problems = n_problems > 0 ? n_problems : 1;
    int64_t cap = 2 * kComputeUnits / problems;
    if (cap > limit) cap = limit;
    if (cap < 1) cap = 1;
    const bool small_tail = rows > 0 && tail_rows <= kMinChunk;
    const int64_t tiles = ((small_tail ? rows : rows + tail_rows) + 31) / 32;
    auto rounds = [&](int64_t n) { return (tiles + 4 * n - 1) / (4 * n); };
    auto fewest = [&](int64_t upto) { int64_t n = upto; while (n > 1 && rounds(n - 1) == rounds(upto)) --n; return n; };
    *tail_own = (small_tail && cap > 1 && rounds(cap - 1) == rounds(cap)) ? 1 : 0;
    const int64_t n = fewest(*tail_own ? cap - 1 : cap);
    // (the tail's workgroups would be the only ones beyond one per compute unit: they wait for a unit to come free)
    if (*tail_own && n * problems <= kComputeUnits && (n + 1) * problems > kComputeUnits) *tail_own = 0;
    return (int)n;
}

constexpr int kTagDataRows = 43;          // a head's 128 output dims as rows of three (the last one holds two) ...
constexpr int kTagRowsPerHead = kTagDataRows + 1;   // ... plus the row with the chunk's log-sum-exp or (max, sum) (see merge_tagged_heads)
constexpr int kTagSlots = kMergeChunks + 1;   // tagged partial results per (sequence, KV head): the chunks + the tail's own
constexpr int kTagRegionRows = kTagSlots * (kD / 2);   // rows per head of a pair's region: 64 to a partial result (rk_attn_common.h), or 44 of the form above

// The partial step in one tile per workgroup (rk_partial.hip): 4 or 8 wavefronts of 16 rows, nch workgroups per (sequence,
// KV head) for the `rows` of the small cache and `tail` for at most tail_rows rows of the full one; waves = 0: not used.  Its
// workgroups wait for one another, so all have to be resident at once: by registers and LDS that is three workgroups of 8 wavefronts per
// compute unit for groups of up to 4 heads, two beyond, and twice that of 4.  With the trigger (one wavefront more, 7 registers) it is
// two workgroups of 8 + 1 for groups of up to 4 heads and one beyond (beyond that, us per launch, attn_split_kernel / this one: 4 sequences of
// K = 2048, 32 heads over 8: 11.2 / 14.6, 16 of 512: 11.4 / 14.5, K = 4096, 64 over 8: 9.6 / 14.1, 8 of 1024, 28 over 4: 10.2 / 12.7).  4
// wavefronts while that is one workgroup per unit and the
// tails: more of them share the request and the merge; 8 beyond, with half the partial results to write and read.
// Many partial results to a pair and more than two workgroups per unit (33 MB of rows) are better off in longer stretches
// (attn_split_kernel).  us per launch, attn_split_kernel / 4 / 8 wavefronts, 32 heads over 8 unless noted: 256 rows 6.9 / 4.9 / 5.5,
// 1024: 6.7 / 4.8 / 5.9, 2048: 6.5 / 5.6 / 6.0, 4096: 8.4 / 8.3 / 7.9, 6000: 10.0 / - / 9.3, 8192: 11.2 / - / 11.9; 28 over 4, 2048:
// 7.4 / 5.1 / 5.9, 4096: 7.4 / 6.0 / 6.3, 8192: 9.9 / - / 8.5; 2 sequences of 2048: 8.7 / 7.9 / 7.9, of 4096: 11.2 / - / 11.4; 4 of 1024:
// 9.3 / 7.8 / 8.2, of 2048: 12.3 / 16.8 / 11.1, of 2048 and 28 over 4: 10.1 / 9.3 / 8.8; 8 of 1024: 12.1 / 13.8 / 11.1; 16 of 512:
// 12.2 / 14.1 / 10.8, of 1024: 17.7 / 22.9 / 19.0.
struct TileForm { int waves, nch, tail; bool exact; int tiles; bool late; };
// exact: partial results weighed by (max, sum) pairs (rk_attn_common.h): groups beyond 4 over more than 16 pairs, which have no tagged form in
// attn_split_kernel and kept such pairs before they came here; a lane of a wavefront each, and the region has room for 65 rows of each.  us per launch, attn_split_kernel with
// pairs / this kernel with a lambda / with pairs: 28 heads over 4, 6 sequences of K = 512: 8.5 / 5.2 / 5.4, of 2048: 11.2 / 7.7 / 7.7, 8 of 512:
// 8.5 / 5.8 / 5.9, 16 of 256: 8.6 / 6.2 / 6.4, 64 heads over 8, 8 sequences of 256: 8.3 / 6.3 / 6.5.
// The merge is 4 G units, whatever the number of results: with two of them (or three of 8 wavefronts) a wavefront has several in a row, and
// groups of 8, and any over many pairs, are better off with all rows in one or two workgroups of attn_split_kernel (64 heads over 8, K = 64, 3 / 16 / 32
// sequences: 7.0 / 7.2 / 7.3 against 7.4 / 8.2 / 9.4, K = 192, 16: 7.5 against 8.4; 48 over 8, K = 64, 16 / 32: 7.4 / 7.5 against 7.3 / 8.3; 40 over
// 8, K = 96, 32: 7.75 against 8.1; 28 over 4, K = 64, 16: 7.4 against 7.0).
constexpr int kTileExactChunks = 64;
static_assert(kTileExactChunks * (kD / 2 + 1) <= kTagRegionRows, "a pair's region holds them");
static inline TileForm partial_tile_form(int64_t rows, int64_t tail_rows, int64_t problems, int G, bool trig) {
    const bool exact = G > 4 && problems > 16;
    for (int waves = 4; waves <= 8; waves += 4) {
        const int wg = 16 * waves;
        const int64_t nch = (rows + wg - 1) / wg, tail = (tail_rows + wg - 1) / wg, total = (nch + tail) * problems;
        if (exact && nch + tail <= (waves == 4 ? 2 : 3) && (G == 8 || problems >= (G > 5 ? 128 : 192))) continue;
        if (trig && waves == 8 && total > (G > 4 ? 1 : 2) * kComputeUnits) continue;
        if (nch > kMergeChunks || nch + tail > (exact ? kTileExactChunks : kTagSlots)) continue;
        if (waves == 4 ? nch * problems <= kComputeUnits && total <= 2 * kComputeUnits
                       : total <= 2 * kComputeUnits || (G <= 4 && total <= 3 * kComputeUnits && nch <= 20))
            return {waves, (int)nch, (int)tail, exact, 1, false};
    }
    return {0, 0, 0, false, 0, false};
}

// ... with two tiles of 16 rows to each of 8 wavefronts, 256 rows to a workgroup: half the partial results to write and read, for a longer chain ahead of
// them.  The rows since have workgroups of their own, or, where those would be the only ones beyond one per unit, the slots that the small cache's
// rows leave (0.5 - 0.9 us, as they are requested late, against 3 for a second workgroup on some of the units).  `fixed`: every row since takes the place of a
// selected one.
// One workgroup per unit: instead of more than 512 of 128 rows (that are not resident, or three to a unit), or of more than 256 where their results
// are many.  All rows are requested before the lengths are known.  Two per unit, where they come close to filling the units (but for 16 pairs, which
// attn_split_kernel does as well), are bound by memory: rows that a sequence turns out not to hold cost as much as those that it does, and whole
// dies have none of its workgroups.  There, and where the workgroups of a pair are few or many of the rows since may be beside the small cache's, the
// wavefronts' second tiles, the cache's second half, are requested once the lengths are known (`late`): hidden behind the first ones' traffic.
// Time as a ratio of the form before (attn_split_kernel or one tile), rows from memory, K rows cached / half of them: one per unit 0.94 / 0.97 (one tile
// resident), 0.87 / 0.95 (not); two per unit, all at once 0.90 - 0.95 / 1.24, late 0.92 - 0.96 / 1.0; lengths uniform up to K: 1.07 and 0.96.  us per launch, before /
// this: 32 heads over 8, 8192 rows with a fixed size 12.1 / 10.1, 6000 9.2 / 8.5, 4 sequences of 2000 11.9 / 10.2, 8 of 1000 11.6 / 10.3; 28 over 4, 9000 10.5 / 8.7,
// 16000 12.2 / 10.0, 4 of 4000 12.5 / 10.3, 8 of 2000 12.9 / 10.3, 16 of 1000 12.6 / 10.7; 64 over 8, 4 of 2000 12.2 / 10.3; late: 32 over 8, 12 of 1150 16.0 / 14.3; 40 over
// 8, 5 of 3000 17.3 / 16.2; 48 over 8, 3 of 4900 21.6 / 15.9.
static inline TileForm two_tile_form(int64_t rows, int64_t tail_rows, int64_t problems, int G, bool fixed) {
    const TileForm none{0, 0, 0, false, 0, false};
    const bool exact = G > 4 && problems > 16;
    const int64_t all = fixed ? (rows > tail_rows ? rows : tail_rows) : rows + tail_rows;
    const int64_t nch = (rows + 255) / 256, ones = (rows + 127) / 128, one_total = (ones + (tail_rows + 127) / 128) * problems;
    int64_t tail = (tail_rows + 255) / 256;
    if (nch < 2 || tail == 0) return none;
    if ((nch + tail) * problems > kComputeUnits && all <= nch * 256) tail = 0;
    const int64_t total = (nch + tail) * problems;
    if (nch > kMergeChunks || nch + tail > (exact ? kTileExactChunks : kTagSlots) || total > 2 * kComputeUnits) return none;
    if (exact && nch + tail <= 3 && (G == 8 || problems >= (G > 5 ? 128 : 192))) return none;      // (see partial_tile_form)
    const bool better = total <= kComputeUnits ? one_total > 2 * kComputeUnits || (one_total > kComputeUnits && ones >= (G > 4 ? 12 : 40))
                        : one_total > 2 * kComputeUnits && 8 * total >= 7 * 2 * kComputeUnits && nch >= (G == 8 ? 5 : 4) && 2 * tail_rows <= nch * 256 && problems != 16;
    return better ? TileForm{8, (int)nch, (int)tail, exact, 2, total > kComputeUnits || nch <= 3 || (tail == 0 && tail_rows > 256)} : none;
}

static inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kBatchLayers = 32;         // layers one batched launch (rk_refresh_batched) takes; more go in several launches
constexpr int kHistBins = 2048;          // first-level histogram of the selection: top 11 key bits
constexpr int kMaxCandidates = 16384;    // most candidates the fast selection path sorts in LDS
constexpr int kHistShift = 32 - 11;      // key bits below the first-level histogram bin
constexpr int kPoolTile = 512;           // positions one workgroup pools and histograms ...
constexpr int kPoolTileLong = 1024;      // ... over rows of kPoolLongFrom positions or more: there the chip is full
constexpr int kPoolLongFrom = 98304;     // anyway and fewer, larger tiles win (per call at 131072 positions: selection
                                         // 38.2 -> 35.6 us, full step with selection 151.7 -> 144.9; at 32k and 64k
                                         // larger tiles lose: 17.4 -> 18.4 and 21.6 -> 22.2 us)
static inline int pool_tile_for(int64_t max_len) { return max_len >= kPoolLongFrom ? kPoolTileLong : kPoolTile; }

// Candidate slots per (sequence, KV head) of the selection: the K winners plus the rest of the
// histogram bin that holds the K-th score.
static inline int topk_cand_cap(int64_t k) {
    int64_t c = 1024;
    while (c < 2 * k && c < kMaxCandidates) c *= 2;
    return (int)c;
}

// Workgroups that share one row of the selection (a power of two; select_part, rk_topk.hip), for `rows` (sequence, KV head) pairs
// in the launch: 8, as long as all are resident at once (one per compute unit).  us per call of rk_topk_select (pooling included)
// with 1 / 2 / 4 / 8 / 16: 8 rows of 32768, K = 2048: 16.1 / 15.1 / 14.8 / 14.9 / 15.6; of 131072, K = 8192: 35.9 / 25.8 / 24.1 / 23.3 /
// 23.3; of 2048, K = 256: 12.5 / 10.9 / 10.8 / 11.0 / 11.6; 4 rows of 65536, K = 4096: 22.2 / 18.9 / 18.1 / 17.5 / 17.4; 32 rows of
// 65536, K = 8192: 33.4 / 28.0 / 26.6 / 25.8 / 36.7; 64 rows of 8192: 14.7 / 14.3 / 14.0 / 20.3; 128 rows of 16384: 22.2 / 21.9 / 29.9.
// (What this replaced, every row's candidates listed by a workgroup per 4096 positions and ranked by the last to arrive, one
// workgroup alone up to 8192: 16.0, 28.9, 13.4, 17.8, 42.0, 15.3, 32.9.)
static inline int select_parts(int64_t rows) {
    int64_t parts = 8;
    while (parts > 1 && parts * rows > kComputeUnits) parts /= 2;
    return (int)parts;
}

// ---- stretches of scores that the parts of a row's selection take (select_part, rk_topk.hip) ----
// Scores >= 0 as whole numbers (their bits), the first-level histogram's bins of 2^kHistShift of them.  The stretch of part i
// is [B(i + 1), B(i)): B leaves t = i / parts of the K' ranks above it, as the histogram has it and, inside the bin that holds rank t,
// as if its scores thinned out upwards at the rate at which they do from there to the bin above: `at`; `end` is where that bin ends and
// `above` the positions beyond.  Parts that share a bound work it out from the same numbers; ranks are counted, so that a bound
// that is off costs time and no more.
struct StretchBound { uint32_t at, end, above; };
// The bin [end - width, end) holds rank t: `above` positions in higher bins, `h` in this one, above < t <= above + h.
// `ratio`: how many times as dense its lower end is as its upper one.
__host__ __device__ static inline StretchBound stretch_bound(uint32_t t, uint32_t spare, uint32_t end, uint32_t width, uint32_t above, uint32_t h, float ratio) {
    if (t - above == h) return {end - width, end - width, t};      // the whole bin: nothing to count
    // (one thread's work while the others wait: reciprocals as they come; the multiply-add by name, so that every copy of this rounds alike)
#ifdef __HIP_DEVICE_COMPILE__
    float part = (float)(t + spare - above) * __builtin_amdgcn_rcpf((float)h);
    if (ratio > 1.f) part = __builtin_amdgcn_logf(fmaf(part, ratio - 1.f, 1.f)) * __builtin_amdgcn_rcpf(__builtin_amdgcn_logf(ratio));
#else
    float part = (float)(t + spare - above) / (float)h;
    if (ratio > 1.f) part = log2f(fmaf(part, ratio - 1.f, 1.f)) / log2f(ratio);
#endif
    const float down = part * (float)width;
    return {end - (down < (float)width ? (uint32_t)down : width), end, above};
}
// ... of a bin of the first-level histogram, from the bin above, `up` positions: four bins of equal width to an octave, twice that in the next.
__host__ __device__ static inline float density_ratio(uint32_t bin, uint32_t h, uint32_t up) {
    const float d = (bin & 3u) == 3u ? 0.5f * (float)up : (float)up;
#ifdef __HIP_DEVICE_COMPILE__
    const float r = (float)h * __builtin_amdgcn_rcpf(d);
#else
    const float r = (float)h / d;
#endif
    return up == 0 || !(r > 1.25f) ? 1.f : r < 16.f ? r : 16.f;
}
// Ranks by which the last part's estimate goes beyond K'.
__host__ __device__ static inline uint32_t last_spare(uint32_t kprime) { return (kprime * 3u >> 3) + 16u; }
// The lower end that a part starts with.  The last part's is an estimate, `floor` (the K'-th score's bin) what it may have to go down to;
// in a bin of tens of millions of positions that estimate can fall on the part's own upper end `top`, and an empty
// stretch would be taken for one without candidates: all of the bin then.
__host__ __device__ static inline uint32_t stretch_low(uint32_t estimate, uint32_t floor, uint32_t top) {
    return estimate <= floor || estimate >= top ? floor : estimate;
}

// A few long rows are listed by a workgroup per 4096 positions and ranked by the last to arrive instead (select_listed_kernel): parts all read the whole
// row, which takes a CU 40 us per million positions and leaves the chip idle; ranking K positions in one workgroup costs more than
// in eight.  `rows`: (sequence, KV head) pairs in the launch, of all layers where it takes several.  us per call of rk_topk_select, parts / listed, log-normal
// scores: one row of 65537, K = 2730: 18.9 / 16.0, of 131073, K = 2048: 21.5 / 16.4, of 1048576, K = 512: 67 / 33, of 4194304: 236 / 106; 4 rows of
// 65537, K = 4096: 20.4 / 19.1, of 1048576: 84 / 72; 6 of 98305, K = 1536: 21.1 / 18.8; one row of 36001, K = 562: 1.0 of the parts' time; K an eighth of the row: 1.0 to 1.2, a
// twelfth 1.0 to 1.1; 4 rows of 131073, K = 8192, one of 180001, K = 11250: 1.06; 8 rows: 1.0 to 1.45.  Scores in tight clusters, no pooling (crowded buckets to rank): 1.1 to 1.4.
// A full step with the batched refresh, K = 1024, 2 layers of one KV head, 131072 rows: 69.8 / 65.5, 524288: 155.6 / 139.4, 3 layers of 2, 131072:
// 122.1 / 118.2; 12 and 16 rows, 131072 to 1048576: 0.96 to 1.01 of listing with parts.
constexpr int kListRows = 6;
constexpr int64_t kListFrom = 49152;
static inline bool select_listed(int64_t max_len, int64_t k, int64_t rows) {
    const bool few = k <= 4096 || (rows <= 3 && k <= 8192);
    return rows <= (k <= 4096 ? kListRows : 4) && max_len >= kListFrom && max_len >= (few ? 16 : 20) * k;
}

// Device workspace, carved in this order (every region 256-byte aligned).  The regions up to and
// including tag_rows must be zero when a workspace is first used (rk_workspace_init clears the
// whole workspace once); the counters and histograms are left cleared by the kernels that use
// them, the call numbers and tags only ever grow.  Where these regions lie depends on the
// geometry alone, never on max_len or max_k.
//   counters  int32 [B*Hkv][kCounterStride]  one 128-byte line each: arrival ticket of the split attention
//                                            kernel (word 0), the trigger's ticket (1), slices left over
//                                            (2, 3), number of partial results of the last full pass (4)
//   sel_counters int32 [B*Hkv][2]            arrival tickets of the selection (word 0); of its listing form the
//                                            runs listed (0) and the tickets (1)
//   epochs    uint32 [B*Hkv]                 call number of the last merge inside a split kernel
//   hist      uint32 [B*Hkv][kHistBins]      first-level histogram of the pooled scores (added to two bins at a time)
//   tag_rows  16 B  [B*Hkv][kTagSlots][G*64]  tagged partial results of the kernels that merge
//                                            inside the launch (see rk_attn_common.h, and merge_tagged_heads in rk_attn.hip)
//   lse       fp32  [B*Hq]                   log-sum-exp when the caller does not ask for it
//   part_ml   fp32  [B*Hkv][kMaxChunks][G][2] running max and sum of every partial result
//   part_o    fp32  [B*Hkv][nch][G][128]     unnormalised partial outputs
//   pooled    fp32  [B*Hkv][max_len up to a multiple of 4]   group-max, pooled scores of the selection
//   scores    fp32  [B*Hq][max_len up to a multiple of 4]    raw scores between the two kernels of
//                                                            rk_full_attn_select
//   cand_list uint64 [B*Hkv][cand_cap]       (few long rows only) runs of candidates of the selection's listing form
constexpr int kCounterStride = 32;       // int32 between two arrival counters: one 128-byte line each
constexpr int kCountWord = 4;
constexpr int kRaggedMaxBatch = 64;      // most sequences whose workgroups are shared out by length
static inline int ragged_batch_of(const rk_geom* g) { return (g->batch > 1 && g->batch <= kRaggedMaxBatch) ? g->batch : 0; }
struct Workspace {
    int32_t* counters;
    int32_t* sel_counters;
    uint32_t* epochs;
    uint32_t* hist;
    uint32_t* tag_rows;
    float* lse;
    float* part_ml;
    float* part_o;
    float* pooled;
    float* scores;
    uint64_t* cand_list;  // NULL: more rows, or shorter ones, than the listing form takes
    int cand_cap;         // candidate slots the selection sorts in LDS
    int max_chunks;       // nch above
    size_t total;
};

// Row stride of the pooled-score area: rows are read with 16-byte loads.
static inline int64_t pooled_row_stride(int64_t max_len) { return (max_len + 3) / 4 * 4; }

// Bytes of the regions that must be zero at first use (the head of the workspace).
static inline size_t zero_kept_bytes(const rk_geom* g) {
    const size_t problems = (size_t)g->batch * g->n_kv_heads;
    const size_t G = (size_t)(g->n_q_heads / g->n_kv_heads);
    size_t off = align_up(problems * ((size_t)kCounterStride + 2 + 1) * sizeof(int32_t), 256);
    off += problems * kHistBins * sizeof(int32_t);
    return off + problems * kTagRegionRows * G * 16;
}

static inline int max_chunks_for(int64_t max_len) {
    int64_t n = (max_len + kMinChunk - 1) / kMinChunk;
    if (n > kMaxChunks) n = kMaxChunks;
    if (n < 1) n = 1;
    return (int)n;
}

// Workgroups per (sequence, KV head) of the score-emitting split kernel of a full step (the
// finishing kernels must be told the same number).  The launch aims at about four tiles of 32 rows
// per wavefront, in whole multiples of the 256 CUs, between one and four workgroups per CU.
// Measured on the kernel alone, total workgroups -> us per launch (8 KV heads unless noted):
//   32778 rows:            256 -> 25.8, 512 -> 24.8 - 25.2, 768 -> 25.7 - 26.2, 1024 -> 25.6 - 25.7
//   65546 rows, 4 heads:   256 -> 28.5, 512 -> 27.6, 768 -> 28.6 - 28.9, 1024 -> 29.0 - 29.4
//   131082 rows:           256 -> 103.0, 512 -> 102.4 - 102.9, 768 -> 102.5, 1024 -> 100.1
// (384 workgroups, uneven over the CUs: 28.8 / 32.8 / 115.3.)  Few tiles per wavefront leave the
// launch's fixed costs (start, the merge across the wavefronts, the partial results) a larger share
// and make a ragged last round (2.67 tiles per wavefront with 768 workgroups at 32k rows) cost more;
// long rows want more loads in flight.  768 workgroups are left out: for groups of 4 heads (170 registers) the kernel is resident
// twice per CU, and they would be one and a half rounds (one layer with its selection, 768 -> 512: 2 sequences of 24000
// rows 58.7 -> 55.6 us, one of 50000 60.9 -> 56.7).  For the other groups (168 registers, three per CU) they would be
// one round, and it makes no difference (one sequence, 768 / 512: 50000 rows of 8 KV heads, groups of 1, 2 and 8: 53.2 / 53.0,
// 54.9 / 54.1, 63.0 / 63.0; 100000 rows of 4 KV heads, groups of 7: 62.3 / 62.3).
static inline int emit_split_target(const rk_geom* g, int64_t max_len) {
    const int64_t tiles = (max_len + 31) / 32 * g->batch * g->n_kv_heads;
    int64_t target = (tiles / 16 + kComputeUnits / 2) / kComputeUnits * kComputeUnits;      // 16 tiles per workgroup: 4 per wavefront
    if (target < kComputeUnits) target = kComputeUnits;
    if (target > 2 * kComputeUnits) target = (target < 4 * kComputeUnits ? 2 : 4) * kComputeUnits;
    return (int)target;
}
static inline int emit_split_workgroups(const rk_geom* g, int64_t max_len) {
    return split_workgroups(max_len, (int64_t)g->batch * g->n_kv_heads, kMaxChunks, emit_split_target(g, max_len));
}

// The attention of an H2O step over budget + 1 rows: the same aim, 768 workgroups among the choices (that kernel is
// resident three times per CU).
static inline int h2o_split_workgroups(const rk_geom* g, int64_t max_rows) {
    const int64_t problems = (int64_t)g->batch * g->n_kv_heads;
    int64_t target = ((max_rows + 31) / 32 * problems / 16 + kComputeUnits / 2) / kComputeUnits * kComputeUnits;
    if (target < kComputeUnits) target = kComputeUnits;
    if (target > 4 * kComputeUnits) target = 4 * kComputeUnits;
    return split_workgroups(max_rows, problems, kMaxChunks, (int)target);
}

// Workgroups per (sequence, KV head) of the same kernel where it merges its partial results itself (nothing but the
// output merge would follow it): no more than there are slots for; groups of more than 4 heads, whose merge by the last
// arrival takes two heads per wavefront, stay with one residency round of 512 workgroups, merged by slices.  Full
// step, us per layer at 768 or 1024 -> 512 workgroups: 6 ragged sequences of 10k rows, 4 KV heads of 7: 57.4 -> 47.7; 2 of
// 24000 rows, 8 of 4: 64.7 -> 53.6; 16 ragged of 5.5k rows, 4 of 7: 89.7 -> 82.9; 16 ragged of 10k, 8 of 4, stays with
// 1024: 186.0 against 188.4.
// 0: compute units would be left without work (few pairs with long rows, small batches), and the merge stays a launch of
// its own.  (That the pairs do not divide 256 is no reason: one sequence of 5 KV heads, 16384 rows, 255 workgroups 13.2 us,
// with the merge launch 15.5; 3 sequences of 8 KV heads, 8000 rows, 240 workgroups 22.4 against 25.4.)
// Where the 64 slots bind, a total between 256 and 512 would leave some CUs a workgroup more than others, and one beyond 512
// start a second residency round that is merged by the last arrival: 256 or 512 then, as near as the pairs come (us per
// deferred step with the merge launch, with 64 partial results to a pair, as here: 3 sequences of 131072 rows, 4 KV heads of 4,
// 768 -> 504 workgroups: 162.4, 166.9, 147.2; 3 KV heads, 576 -> 504: 123.5, 126.6, 112.2; 2 sequences of 65536 rows, 8 KV
// heads, 1024 -> 512: 108.3, 109.1, 103.3; one sequence, 5 KV heads, 320 -> 255: 69.9, 71.6, 62.2; 7 KV heads, 448 ->
// 252: 93.7, 90.8, 86.3).
// A ragged batch with one or two KV heads: one sequence much longer than the others would have to make do with 64 or 128
// workgroups in all, while the launch it replaces gives it 256 of the CUs (us per deferred step with the merge launch before
// these forms, merged inside, with it now: one of 131072 rows and 3 of 64, one KV head: 24.2, 29.0, 21.7; and 15 of 64, two KV
// heads: 36.7, 37.9, 32.6; sequences alike, 16 of 65536, one KV head: 111.5, 105.4, 102.7; three KV heads, 131072 and 15 of
// 64, stay inside: 53.9, 44.2, 47.6).
static inline int inside_split_workgroups(const rk_geom* g, int64_t max_len) {
    const int64_t problems = (int64_t)g->batch * g->n_kv_heads;
    if (ragged_batch_of(g) != 0 && max_len > (int64_t)kMergeChunks * kMinChunk && kMergeChunks * g->n_kv_heads <= kComputeUnits / 2) return 0;
    int target = emit_split_target(g, max_len);
    if (target > 2 * kComputeUnits && g->n_q_heads > 4 * g->n_kv_heads) target = 2 * kComputeUnits;
    int n = split_workgroups(max_len, problems, kMergeChunks, target);
    if (n == kMergeChunks) {
        const int64_t total = n * problems, round = 2 * kComputeUnits;
        if (total > round) n = (int)(round / problems);
        else if (total > kComputeUnits && total < round) n = (int)(kComputeUnits / problems);
    }
    if ((g->batch > 1 || max_len > (int64_t)kMergeChunks * kMinChunk) && (n + 1) * problems <= kComputeUnits) return 0;
    return n;
}
// Deferred full steps whose merge inside weighs the partial results by their fp32 log-sum-exps, as a partial step does
// (|lse| * 2^-24 to a weight), instead of exactly as the merge launch (see merge_tagged_heads): groups of up to 4 heads,
// rows shared out alike, one residency round at 4 tiles per wavefront.  The exact form takes 0.6 us longer in that one
// launch (32 layers of 33k rows 1028 -> 1046 us per step).
static inline bool merges_in_fp32(const rk_geom* g, int64_t max_len) {
    const int64_t problems = (int64_t)g->batch * g->n_kv_heads, n = inside_split_workgroups(g, max_len);
    return g->n_q_heads <= 4 * g->n_kv_heads && ragged_batch_of(g) == 0 && (max_len + 31) / 32 * problems < 40 * kComputeUnits &&
           n * problems <= 2 * kComputeUnits && n == emit_split_workgroups(g, max_len);
}

// ... and of a full step whose pooling is deferred: the pooling kernels must be told the same number.
static inline int deferred_split_workgroups(const rk_geom* g, int64_t max_len) {
    const int inside = inside_split_workgroups(g, max_len);
    return inside > 0 ? inside : emit_split_workgroups(g, max_len);
}

// A trigger's test step in one launch (test_step_kernel): over one sequence, where its full pass merges inside and its partial step fits 4 wavefronts to
// a workgroup, of 16 rows each or of two tiles of 16, and all workgroups of either are resident at once (two per compute unit).  With several
// sequences a workgroup of one would have to wait for the decisions of the others.  us per layer of a test step (its share of the batched refresh included), two
// launches / one, none full and all full: 65536 rows, K = 4096, 28 heads over 4: 9.9 / 7.6 and 42.9 / 38.8; 32768, 2048, 32 over 8: 9.7 / 7.2, 40.9 / 39.8;
// 8192, 700, 32 over 8: 8.1 / 6.2, 18.8 / 17.1; 3000, 256, 28 over 4: 8.2 / 6.2, 14.2 / 12.1; 16384, 1000, 16 over 4: 7.9 / 5.8, 18.5 / 17.1; in two tiles (and
// where the bound on the rows since, which the trigger's schedule lets grow, leaves no slot for a 66th result), 32 over 8: 40000, 3000: 10.4 / 8.9, 47.2 / 46.0;
// 60000, 4096: 12.9 / 10.1, 65.9 / 65.1; 65536, 7000: 14.9 / 13.2, 78.7 / 73.6; 64 over 8, 40000, 3500: 12.0 / 10.9, 54.4 / 53.7.
static inline TileForm test_step_form(const rk_geom* g, int64_t n_sel, int64_t max_recent, int64_t max_len) {
    if (g->batch != 1) return {0, 0, 0, false, 0, false};
    const int64_t inside = inside_split_workgroups(g, max_len);
    if (inside == 0 || inside * g->n_kv_heads > 2 * kComputeUnits || (g->n_kv_heads > 16 && g->n_q_heads > 4 * g->n_kv_heads)) return {0, 0, 0, false, 0, false};
    for (int tiles = 1; tiles <= 2; ++tiles) {             // 64 or 128 rows to a workgroup
        const int64_t wg = 64 * tiles, nch = (n_sel + wg - 1) / wg, tail = (max_recent + wg - 1) / wg;
        if (nch <= kMergeChunks && nch + tail <= kTagSlots && (nch + tail) * g->n_kv_heads <= 2 * kComputeUnits &&
            (tiles == 2 || nch * g->n_kv_heads <= kComputeUnits)) return {4, (int)nch, (int)tail, false, tiles};
    }
    return {0, 0, 0, false, 0, false};
}

// Form and split of the two passes of rk_window_select over K (see rk_window.hip): 16 T rows per wavefront and step,
// wg_rows per workgroup and step, nch workgroups per (sequence, KV head), at most `limit`.
// T = 4 takes 512 rows per workgroup and round and gains from every block of columns it holds the rows for, but a last round
// with little in it costs as much as a full one; T = 2, 128 rows at a time, does not care.  Up to 2 blocks T = 2, from 9 on T
// = 4; between, T = 4 where the rows fill 17/20 of its rounds (of the chip's up to 4 blocks: there fewer, longer workgroups gain
// nothing either).  Whole call, us, 32 heads over 8, both passes with 32 rows and masks everywhere / T = 4 / T = 2: 16 queries (4
// blocks): 24000 rows 57.3 / 55.7 / 52.3, 36000 70.2 / 77.9 / 65.4, 64000 95.3 / 87.4 / 90.1, 66000 96.4 / 98.5 / 91.5; 24 queries (6):
// 16000 53.3 / 47.0 / 49.2, 36000 76.1 / 80.6 / 68.7, 80000 117.9 / 111.4 / 108.5; 32 queries (8): 32768 89.3 / 67.5 / 71.7, 36000
// 90.6 / 85.8 / 74.5, 57000 127.6 / 101.2 / 103.2, 100000 168.1 / 144.7 / 137.2; 28 heads over 4, 8 queries (4): 76000 72.3 / 80.1 / 68.1;
// 64 over 8, 20 queries (10): 36000 105.1 / 103.6 / 91.9, 58000 137.7 / 112.4 / 119.6, 32 queries (16): 36000 166.9 / 131.8 / 145.4.
constexpr int kWinTargetWgs = 512;     // workgroups of eight wavefronts a pass aims for: two per CU
struct WindowForm { int T, wg_rows, nch; };
static inline WindowForm window_form(int64_t max_rows, int64_t problems, int column_blocks, int limit) {
    const bool few = max_rows * problems <= (int64_t)kWinTargetWgs * 128;
    WindowForm f = few ? WindowForm{1, 128, 1} : WindowForm{4, 512, 1};
    int64_t per = kWinTargetWgs / problems;
    if (per < 1) per = 1;
    const int64_t stretches = (max_rows + f.wg_rows - 1) / f.wg_rows;
    f.nch = (int)(per < stretches ? per : stretches);
    if (f.nch > limit) f.nch = limit;
    if (few || column_blocks > 8) return f;
    const int64_t round = (column_blocks <= 4 ? per : f.nch) * f.wg_rows, rounds = (max_rows + round - 1) / round;
    if (column_blocks > 2 && 20 * max_rows >= 17 * rounds * round) return f;
    return {2, 128, split_workgroups(max_rows, problems, limit)};
}

static inline Workspace carve(const rk_geom* g, int64_t max_len, int64_t max_k, void* base) {
    Workspace w;
    const size_t problems = (size_t)g->batch * g->n_kv_heads;
    const size_t G = (size_t)(g->n_q_heads / g->n_kv_heads);
    w.max_chunks = max_chunks_for(max_len);
    char* p = (char*)base;
    size_t off = 0;
    w.counters = (int32_t*)(p + off); off += problems * kCounterStride * sizeof(int32_t);
    w.sel_counters = (int32_t*)(p + off); off += 2 * problems * sizeof(int32_t);
    w.epochs = (uint32_t*)(p + off);  off += problems * sizeof(uint32_t);
    off = align_up(off, 256);
    w.hist = (uint32_t*)(p + off);    off += problems * kHistBins * sizeof(uint32_t);
    w.tag_rows = (uint32_t*)(p + off); off += problems * kTagRegionRows * G * 16;
    w.lse = (float*)(p + off);        off += align_up((size_t)g->batch * g->n_q_heads * sizeof(float), 256);
    w.part_ml = (float*)(p + off);    off += align_up(problems * kMaxChunks * G * 2 * sizeof(float), 256);
    w.part_o = (float*)(p + off);     off += align_up(problems * w.max_chunks * G * kD * sizeof(float), 256);
    w.pooled = (float*)(p + off);     off += align_up(problems * (size_t)pooled_row_stride(max_len > 0 ? max_len : 1) * sizeof(float), 256);
    w.scores = (float*)(p + off);     off += align_up((size_t)g->batch * g->n_q_heads * (size_t)pooled_row_stride(max_len > 0 ? max_len : 1) * sizeof(float), 256);
    w.cand_cap = topk_cand_cap(max_k > 0 ? max_k : 1);
    w.cand_list = nullptr;
    if (problems <= (size_t)kListRows && max_len >= kListFrom) {
        w.cand_list = (uint64_t*)(p + off); off += align_up(problems * (size_t)w.cand_cap * sizeof(uint64_t), 256);
    }
    w.total = off;
    return w;
}

static inline int check_geom(const rk_geom* g) {
    if (!g) return RK_ERR_INVALID_ARG;
    if (g->batch <= 0 || g->n_q_heads <= 0 || g->n_kv_heads <= 0) return RK_ERR_INVALID_ARG;
    if (g->n_q_heads % g->n_kv_heads != 0) return RK_ERR_INVALID_ARG;
    if (g->head_dim != kD) return RK_ERR_UNSUPPORTED;
    if (g->n_q_heads / g->n_kv_heads > RK_MAX_GROUP) return RK_ERR_UNSUPPORTED;
    if (g->batch > 65535 || g->n_kv_heads > 65535) return RK_ERR_UNSUPPORTED;
    return RK_OK;
}

static inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

static inline int check_kv(const rk_kv& c, bool need_v = true) {
    if (!c.k || (need_v && !c.v)) return RK_ERR_INVALID_ARG;
    if (!aligned16(c.k) || !aligned16(c.v)) return RK_ERR_INVALID_ARG;
    // row indices are int32 and the kernels step past the end by up to kMaxChunks * kMinChunk rows
    if (c.stride_b < 0 || c.stride_h < 0 || c.capacity <= 0 || c.capacity > INT32_MAX - 2 * kMaxChunks * kMinChunk) return RK_ERR_INVALID_ARG;
    if (c.stride_b % 8 != 0 || c.stride_h % 8 != 0) return RK_ERR_INVALID_ARG;
    if (c.stride_b >= (1ll << 56)) return RK_ERR_UNSUPPORTED;   // the top byte of the sequence stride travels as a flag to the kernels
    if (c.stride_h > INT32_MAX) return RK_ERR_UNSUPPORTED;      // the head stride travels as 32 bits to the kernels
    return RK_OK;
}

static inline int check_workspace(const rk_geom* g, int64_t max_len, int64_t max_k, void* ws,
                                  size_t bytes, Workspace* out) {
    if (!ws || ((uintptr_t)ws & 255u) != 0) return RK_ERR_WORKSPACE;
    *out = carve(g, max_len, max_k, ws);
    if (bytes < out->total) return RK_ERR_WORKSPACE;
    return RK_OK;
}

static inline int launch_status() {
    return hipGetLastError() == hipSuccess ? RK_OK : RK_ERR_HIP;
}

// Stages shared by the entry points (arguments already checked by the caller).
//   full_attn_stage: the split kernel, then either the merge inside it (no weights), the merge +
//     normalise kernel (weights in place), or, with pool_half >= 0, the fused finish that also
//     leaves the pooled group scores and their histogram in the workspace.  no_v: the split kernel
//     is the scores-only one (K rows only; out must be NULL, pool_half >= 0).  defer_pool (with
//     pool_half >= 0 and out != NULL): only the output is finished; the raw scores and the chunk
//     statistics stay in the workspace for pool_batched_stage, which does for several layers at
//     once what the finishing kernel's pooling tiles do for one.  nch: workgroups per (sequence, KV head), where the
//     caller's own rule decides (with weights; 0: this stage's).
//   select_stage: top-K over the pooled scores and histogram that are in the workspace.
__attribute__((visibility("hidden")))
int full_attn_stage(const rk_geom* geom, const void* q, rk_kv full, const int32_t* seq_lens, int32_t max_len,
                    void* out, float* weights, int64_t w_stride, float* lse, const int32_t* pred, int32_t pred_val,
                    const Workspace& ws, hipStream_t st, bool scores_only, int pool_half, bool no_v, int agg,
                    bool defer_pool = false, int nch = 0);
__attribute__((visibility("hidden")))
int pool_batched_stage(const rk_geom* geom, int n_layers, const Workspace* wss, const int32_t* seq_lens, int32_t max_len,
                       int64_t full_capacity, int pool_half, int agg, const int32_t* const* pred, int32_t pred_val,
                       hipStream_t st);
//   gather_attn_stage: rk_gather_attn plus an optional per-sequence count of refreshes.
__attribute__((visibility("hidden")))
int gather_attn_stage(const rk_geom* geom, const void* q, rk_kv full, const int32_t* idx, int32_t k, rk_kv small, const int32_t* seq_lens,
                      int32_t* tail_start, int32_t* n_refresh, void* out, const int32_t* pred, int32_t pred_val, void* workspace,
                      size_t workspace_bytes, hipStream_t st);
//   test_step_stage: a layer's step on which the trigger is tested: rk_partial_attn_triggered, then rk_full_attn_deferred under the
//     decision, in one launch where that has a form.
__attribute__((visibility("hidden")))
int test_step_stage(const rk_geom* geom, const void* q, const rk_layer_state& layer, const rk_schedule* sched, const int32_t* seq_lens, int32_t max_len,
                    int32_t max_recent, void* out, void* workspace, size_t workspace_bytes, hipStream_t st);
//   h2o_attn_stage: the attention of an H2O step, scores and partial results left in the workspace.
__attribute__((visibility("hidden")))
int h2o_attn_stage(const rk_geom* geom, const void* q, const rk_h2o_state& st, const void* k_new, const void* v_new,
                   int32_t budget, const Workspace& ws, hipStream_t stream);
//   gather_stage: rk_gather_small_kv plus an optional per-sequence count of refreshes.
__attribute__((visibility("hidden")))
int gather_stage(const rk_geom* geom, rk_kv full, const int32_t* idx, int32_t k, rk_kv small,
                 const int32_t* seq_lens, int32_t* tail_start, int32_t* n_refresh,
                 const int32_t* pred, int32_t pred_val, hipStream_t stream);
//   pool_stage: group aggregation, max-pool and histogram of normalised per-head scores (first
//     kernel of rk_topk_select); check_select_args: the limits on k, pool_w and agg.
__attribute__((visibility("hidden")))
int pool_stage(const rk_geom* geom, const float* weights, int64_t w_stride, const int32_t* seq_lens,
               int32_t max_len, int32_t pool_w, int32_t agg, const int32_t* pred, int32_t pred_val,
               const Workspace& ws, hipStream_t st);
__attribute__((visibility("hidden")))
int check_select_args(int32_t k, int32_t pool_w, int32_t agg, int32_t max_len);
__attribute__((visibility("hidden")))
int select_stage(const rk_geom* geom, const int32_t* seq_lens, int32_t max_len, int32_t k, int32_t* idx,
                 float* sel_scores, const int32_t* pred, int32_t pred_val, const Workspace& ws, hipStream_t st);

// Batched forms for rk_refresh_batched: the selections, then the gathers, of up to kBatchLayers
// layers in one launch each.  wss[l] holds what rk_full_attn_pool left for layer l.
__attribute__((visibility("hidden")))
int select_batched_stage(const rk_geom* geom, int n_layers, const Workspace* wss, int32_t* const* idx,
                         const int32_t* seq_lens, int32_t max_len, int32_t k, const int32_t* const* pred, int32_t pred_val,
                         hipStream_t st);
__attribute__((visibility("hidden")))
int gather_batched_stage(const rk_geom* geom, int n_layers, const rk_kv* full, const rk_kv* small, int32_t* const* idx,
                         int32_t k, const int32_t* seq_lens, int32_t* const* tail_start, int32_t* const* n_refresh,
                         const int32_t* const* pred, int32_t pred_val, hipStream_t st);

}  // namespace rk
