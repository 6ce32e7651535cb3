// The partial step in one tile per workgroup: partial_tile_kernel.
//
// What bounds it is not the 8 MB of rows of a step (2.6 us for a kernel that only reads them) but a chain: a
// wavefront alone on its SIMD executes an instruction every 8 to 12 cycles, and a launch is requests, one tile, one
// exchange between workgroups.  attn_split_kernel gives a wavefront 32 rows and all 128 dims of the output, so that four partial
// outputs have to be rescaled and added through LDS before anything is published.  Here
//   - a wavefront has 16 rows of S^T = K Q^T: half the loads, exponentials and packing;
//   - the wavefronts agree on the maximum and exchange P through LDS, and each then works out O for its own 16 or 32 dims
//     over all the rows: nothing is left to add up, and no accumulator is rescaled;
//   - O^T = V^T P^T leaves four consecutive dims of one head in a lane: two rows { x, x, lambda, tag } to publish, straight
//     from the accumulators, and every row that is read brings the lambda that weighs it;
//   - the kernel's scalars are read in one round trip, behind nothing and ahead of the rows.
// us per launch, one sequence, 32 heads over 8: K = 256: 6.9 -> 4.9, 1024: 6.7 -> 4.8, 2048: 6.5 -> 5.6, 4096: 8.4 -> 7.9; 28 over 4, K
// = 4096: 7.4 -> 6.0 (more at partial_tile_form).  At K = 2048 in cycles after a wavefront's first instruction: first rows
// there 3700, S^T 3800, maximum known 4000, P and V in LDS 4800, O 5300, published 5800, merged 9500 (the slowest workgroups
// start 0.3 us after the first); the launch to launch time is 1.2 us more than the slowest of it.  The latency is paid for in traffic: 64 rows
// of 16 bytes per head and partial result instead of 44, and twice the partial results (K = 2048: 12.0 MB per launch against 9.8
// with attn_split_kernel, 8.4 needed), which is one reason why more than two workgroups per unit are better off there.
//
// Longer small caches and batches: two tiles to a wavefront (two_tile_form has the figures).  16 sequences of 1000 or one of 8192 rows are 67 and 33 MB, which
// take 11 and 5.5 us to arrive; half as many partial results is what is gained, with P's lanes beyond the group left out of LDS so that two workgroups of
// 256 rows fit a compute unit.  LATE: with two per unit the second tiles' requests can wait for the lengths behind the first ones' traffic (2 % of the launch), so
// that rows which a sequence does not hold are not read.
#include "rk_tile.h"

namespace rk {

static_assert(sizeof(TileParams) == 136, "arguments");

template <int G, int NW, bool TRIG, bool EXACT, int R, bool LATE>
__global__ __launch_bounds__((NW + TRIG) * 64, 4)
void partial_tile_kernel(const uint16_t* k1, const uint16_t* v1, int64_t s_b_and_tail, int32_t s_h, uint32_t rows_heads,
                         const int32_t* seq_lens, const int32_t* tail_start, const uint16_t* q, const TileParams p) {
    partial_tile<G, NW, TRIG ? kTestBeside : kNoTest, EXACT, false, R, 0, LATE>(k1, v1, s_b_and_tail, s_h, rows_heads, seq_lens, tail_start, q, p, blockIdx.x, blockIdx.y, blockIdx.z);
}

// The step right after a selection, with the gather in it: bound by memory, every row read and written once, where a gather writes what a second
// launch then reads.  Whole rows of K through LDS: K = 8192, 32 heads over 8: 18.0 us with K loaded straight into the operand layout, 17.0.  us,
// gather + step / this one, 32 heads over 8 unless noted: K = 256: 7.9 / 5.9, 2048: 10.5 / 7.0, 4096: 14.9 / 9.8, 6000: 17.9 / 13.4, 8192:
// 24.1 / 17.0; 28 over 4, 4096: 11.1 / 7.4; 4 sequences of 1024: 14.9 / 9.7, of 2048: 24.2 / 16.0; 64 over 8, 4 of 700: 13.0 / 8.5.
template <int G, int NW, bool EXACT>
__global__ __launch_bounds__(NW * 64, 4)
void gather_tile_kernel(uint16_t* k1, uint16_t* v1, int64_t s_b_and_tail, int32_t s_h, uint32_t rows_heads,
                        const int32_t* seq_lens, const int32_t* idx, const uint16_t* q, const TileParams p) {
    partial_tile<G, NW, kNoTest, EXACT, true>(k1, v1, s_b_and_tail, s_h, rows_heads, seq_lens, idx, q, p, blockIdx.x, blockIdx.y, blockIdx.z);
}

template <int G, int NW, bool EXACT, int R = 1, bool LATE = false>
static int launch_g(const AttnParams& p, int batch, bool trig, const int32_t* idx, hipStream_t st) {
    const TileArgs a = tile_args(p);
    dim3 grid(p.nch + p.tail_wg, p.Hkv, batch);
    if constexpr (R > 1) {
        hipLaunchKernelGGL((partial_tile_kernel<G, NW, false, EXACT, R, LATE>), grid, dim3(NW * 64), 0, st, p.k1, p.v1, a.s_b_and_tail, (int32_t)p.s1_h,
                           a.rows_heads, p.seq_lens, p.tail_start, p.q, a.t);
        return launch_status();
    }
    if (idx != nullptr) {
        hipLaunchKernelGGL((gather_tile_kernel<G, NW, EXACT>), grid, dim3(NW * 64), 0, st, const_cast<uint16_t*>(p.k1), const_cast<uint16_t*>(p.v1),
                           a.s_b_and_tail, (int32_t)p.s1_h, a.rows_heads, p.seq_lens, idx, p.q, a.t);
        return launch_status();
    }
    auto kernel = trig ? partial_tile_kernel<G, NW, true, EXACT, 1, false> : partial_tile_kernel<G, NW, false, EXACT, 1, false>;
    hipLaunchKernelGGL(kernel, grid, dim3((NW + (trig ? 1 : 0)) * 64), 0, st, p.k1, p.v1, a.s_b_and_tail, (int32_t)p.s1_h, a.rows_heads,
                       p.seq_lens, p.tail_start, p.q, a.t);
    return launch_status();
}

template <int G>
static int launch_form(const AttnParams& p, int batch, const TileForm& form, bool trig, const int32_t* idx, hipStream_t st) {
    if (form.tiles == 2) {
        if (trig || idx != nullptr || form.waves != 8) return RK_ERR_UNSUPPORTED;
        if constexpr (G > 4)
            if (form.exact) return form.late ? launch_g<G, 8, true, 2, true>(p, batch, false, nullptr, st) : launch_g<G, 8, true, 2>(p, batch, false, nullptr, st);
        return form.late ? launch_g<G, 8, false, 2, true>(p, batch, false, nullptr, st) : launch_g<G, 8, false, 2>(p, batch, false, nullptr, st);
    }
    if constexpr (G > 4)
        if (form.exact) return form.waves == 4 ? launch_g<G, 4, true>(p, batch, trig, idx, st) : launch_g<G, 8, true>(p, batch, trig, idx, st);
    return form.waves == 4 ? launch_g<G, 4, false>(p, batch, trig, idx, st) : launch_g<G, 8, false>(p, batch, trig, idx, st);
}

int launch_partial_tile(const AttnParams& p, int batch, int G, const TileForm& form, bool trig, const int32_t* idx, hipStream_t st) {
    switch (G) {
#define RK_CASE(g) case g: return launch_form<g>(p, batch, form, trig, idx, st);
        RK_CASE(1) RK_CASE(2) RK_CASE(3) RK_CASE(4) RK_CASE(5) RK_CASE(6) RK_CASE(7) RK_CASE(8)
#undef RK_CASE
        default: return RK_ERR_UNSUPPORTED;
    }
}

}  // namespace rk
