"""Host logic that sizes the launches (csrc/rk_internal.h), checked without a GPU.

A small host program that includes the library's own header is compiled with hipcc and prints what
the rules give for a table of shapes; the test checks the bounds every kernel relies on (at least
one workgroup, never more partial results than the merge has slots for, never more than there are
stretches of 128 rows) and the choices the measurements in the header's comments led to.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2411_05787_amd", "csrc")

PROGRAM = r"""
#include "rk_internal.h"
#include <cstdio>
using namespace rk;
int main() {
    const long rows[] = {1, 100, 128, 129, 512, 1024, 2048, 4096, 8192, 16384};
    const long problems[] = {1, 4, 8, 16, 24, 32, 64, 128, 256, 512, 4096};
    for (long r : rows) for (long p : problems) for (int tail : {0, 10, 128, 500})
        printf("merged %ld %d %ld %d %d %d\n", r, tail, p, merged_split_workgroups(r, tail, p, false),
               merged_split_workgroups(r, tail, p, true), (int)two_batches_pay(r, tail, p));
    for (long r : rows) for (long p : problems) for (int tail : {0, 10, 500}) {
        int own = -1;
        const int n = batched_tagged_workgroups(r, tail, &own, p);
        printf("batched %ld %d %ld %d %d\n", r, tail, p, n, own);
    }
    for (long r : {1L, 100L, 128L, 1024L, 2048L, 3072L, 4096L, 6144L, 8192L, 12288L, 16384L, 100000L}) for (long p : {1L, 4L, 8L})
        for (int tail : {0, 10, 128, 500}) {
            int own = -1;
            const int n = sliced_split_workgroups(r, tail, &own, p, 64);
            printf("sliced %ld %d %ld %d %d\n", r, tail, p, n, own);
        }
    for (long r : {0L, 1L, 64L, 65L, 256L, 700L, 1024L, 2048L, 4096L, 6000L, 8192L, 8193L, 100000L}) for (long p : {1L, 4L, 8L, 12L, 32L, 64L, 128L, 512L, 4096L})
        for (int tail : {0, 1, 64, 65, 128, 500, 100000}) for (int G : {1, 4, 5, 8}) {
            if (r + tail == 0) continue;
            for (int trig = 0; trig < 2; ++trig) {
                const TileForm f = partial_tile_form(r, tail, p, G, trig != 0);
                printf("tile %ld %ld %d %d %d %d %d %d %d\n", r, p, tail, G, trig, f.waves, f.nch, f.tail, (int)f.exact);
            }
        }
    for (long r : {0L, 1L, 256L, 500L, 1000L, 1700L, 2000L, 2048L, 3000L, 4000L, 6000L, 8150L, 8181L, 8192L, 9000L, 16000L, 16384L, 20000L}) for (long p : {1L, 4L, 8L, 16L, 32L, 64L, 128L, 512L})
        for (int tail : {0, 1, 11, 256, 257, 9000}) for (int G : {1, 4, 5, 8}) for (int fixed : {0, 1}) {
            const TileForm f = two_tile_form(r, tail, p, G, fixed != 0);
            printf("two %ld %ld %d %d %d %d %d %d %d %d %d\n", r, p, tail, G, fixed, f.waves, f.nch, f.tail, (int)f.exact, f.tiles, (int)f.late);
        }
    for (long p : {1L, 4L, 8L, 12L, 32L, 33L, 64L, 65L, 128L, 129L, 256L, 257L, 100000L}) printf("parts %ld %d\n", p, select_parts(p));
    for (long l : {1000L, 49151L, 49152L, 65536L, 131072L, 163840L, 196608L, 1000000L}) for (long k : {1L, 3072L, 3073L, 4097L, 8192L, 12288L, 16384L}) for (int b : {1, 2}) for (int hkv : {1, 2, 3, 4, 7}) {
        rk_geom g{b, hkv, hkv, 128, 1.0f};
        const Workspace w = carve(&g, l, k, nullptr), shorter = carve(&g, l - 1, k, nullptr), fewer = carve(&g, l, k - 1, nullptr);
        printf("listed %ld %ld %d %d %d %d\n", l, k, b * hkv, (int)select_listed(l, k, b * hkv), (int)(w.cand_list != nullptr),
               (int)(shorter.total <= w.total && fewer.total <= w.total));
    }
    // the parts of a row whose K' ranks end in a bin of h positions, `above` of the ranks in higher bins: stretches from the top
    // down to where the last part starts, or may have to go down to
    for (long h : {1L, 2L, 3L, 7L, 8L, 100L, 5000L, 100000L, 1L << 21, 20000000L, 40000000L, 60000000L, 100000000L, 1L << 28}) for (int lg : {1, 2, 3}) {
        long open = 0, order = 0, empty = 0;
        for (float ratio : {1.f, 2.f, 16.f}) for (uint32_t above : {0u, 1u, 13u, 4096u}) for (uint32_t k = above + 1; k <= above + h && k <= 16384; k += k < above + 300 ? 1 : 97) {
            const uint32_t width = 1u << kHistShift, floor = (1500u << kHistShift) - 0x80000000u;
            uint32_t upper = floor + width;                       // where the bins above end
            for (int part = 0; part < 1 << lg; ++part) {
                const uint32_t t0 = (k * (uint32_t)part) >> lg, t1 = (k * (uint32_t)(part + 1)) >> lg;
                const bool last = part + 1 == 1 << lg;
                const uint32_t top = t0 > above ? stretch_bound(t0, 0, floor + width, width, above, (uint32_t)h, ratio).at : upper;
                order += top != upper;                            // the stretch above ended there
                if (t1 <= above) continue;
                const uint32_t at = stretch_bound(t1, last ? last_spare(k) : 0u, floor + width, width, above, (uint32_t)h, ratio).at;
                order += at > top || at < floor;
                const uint32_t low = stretch_low(at, last ? floor : at, top);
                open += last && low >= top && low != floor;       // ranks between the stretch and the floor that nobody takes
                empty += last && at >= top && at > floor;
                upper = at;
            }
        }
        printf("stretch %ld %d %ld %ld %ld\n", h, lg, open, order, empty);
    }
    const long lens[] = {1, 2000, 32768, 33008, 65536, 131072, 1000000};
    for (long l : lens) for (int b : {1, 2, 16}) for (int hkv : {1, 4, 8}) {
        rk_geom g{b, hkv * 4, hkv, 128, 1.0f};
        printf("emit %ld %d %d %d\n", l, b, hkv, emit_split_workgroups(&g, l));
    }
    for (long l : {1L, 500L, 2000L, 6000L, 8000L, 8192L, 8193L, 16384L, 20000L, 33008L, 65536L, 100000L, 131072L, 1000000L}) for (int b : {1, 2, 3, 5, 6, 9, 16, 64, 65})
        for (int hkv : {1, 2, 3, 4, 5, 6, 7, 8}) for (int G : {1, 4, 7}) {
            rk_geom g{b, hkv * G, hkv, 128, 1.0f};
            printf("inside %ld %d %d %d %d %d %d %d\n", l, b, hkv, G, inside_split_workgroups(&g, l), emit_split_workgroups(&g, l),
                   deferred_split_workgroups(&g, l), (int)merges_in_fp32(&g, l));
        }
    for (long l : {1L, 50L, 700L, 3000L, 8192L, 33000L, 66000L, 131072L}) for (long k : {64L, 700L, 2048L, 4096L, 8192L}) for (int recent : {1, 64, 65, 500}) for (int b : {1, 2})
        for (int hkv : {1, 3, 4, 8, 16, 32}) for (int G : {1, 4, 7, 8}) {
            rk_geom g{b, hkv * G, hkv, 128, 1.0f};
            const TileForm f = test_step_form(&g, k, recent, l);
            printf("test_step %ld %ld %d %d %d %d %d %d %d %d %d\n", l, k, recent, b, hkv, G, f.waves, f.nch, f.tail, inside_split_workgroups(&g, l), f.tiles);
        }
    for (long l : {1L, 63L, 512L, 513L, 1100L, 1400L, 2100L, 16000L, 32768L, 36000L, 40000L, 64000L, 76000L, 131072L}) for (long p : {1L, 4L, 8L, 128L, 260L, 520L, 4096L})
        for (int blocks : {1, 2, 3, 8, 16}) {
            const int limit = max_chunks_for(l);
            const WindowForm f = window_form(l, p, blocks, limit);
            printf("window %ld %ld %d %d %d %d %d\n", l, p, blocks, limit, f.T, f.wg_rows, f.nch);
        }
    for (long l : {2L, 31L, 128L, 129L, 2049L, 4101L, 8193L, 16701L, 32769L}) for (int b : {1, 4, 16, 70}) for (int hkv : {1, 4, 8}) {
        rk_geom g{b, hkv * 4, hkv, 128, 1.0f};
        printf("h2o %ld %d %d %d %d %d\n", l, b, hkv, h2o_split_workgroups(&g, l), emit_split_workgroups(&g, l), max_chunks_for(l));
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    d = tmp_path_factory.mktemp("sizes")
    src = d / "sizes.cpp"
    src.write_text(PROGRAM)
    exe = d / "sizes"
    # host code only: no offload architecture needed, nothing is launched
    r = subprocess.run([hipcc, "-O1", "-std=c++17", "-I", CSRC, "-x", "hip", "--offload-arch=gfx950", str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr[-2000:]
    rows = [ln.split() for ln in out.stdout.splitlines()]
    return rows


def test_merged_split_bounds(table):
    seen = 0
    for kind, *v in table:
        if kind != "merged":
            continue
        rows, tail, problems, n16, n32, pays = map(int, v)
        counted = rows if tail <= 32 else rows + tail
        stretches = max((counted + 127) // 128, 1)
        for n in (n16, n32):
            assert 1 <= n <= 64
            assert n <= stretches or n == 32, (rows, tail, problems, n)
        if n32 != n16:
            assert n32 == 32 and pays == 1              # the only difference the ticketed form makes
        if pays:
            assert problems <= 8 and rows + (tail if tail > 128 else 0) > 2048
        seen += 1
    assert seen == 10 * 11 * 4


def test_batched_tagged_bounds_and_measured_choices(table):
    got = {}
    for kind, *v in table:
        if kind != "batched":
            continue
        rows, tail, problems, n, own = map(int, v)
        counted = rows if tail <= 128 else rows + tail
        assert own in (0, 1) and 1 <= n <= 64 and n <= max((counted + 127) // 128, 1)
        if tail == 0 or tail > 128:
            assert own == 0
        got[(rows, tail, problems)] = (n, own)
    # the shapes that were measured
    assert got[(2048, 10, 128)] == (2, 0) and got[(1024, 10, 128)] == (2, 0)      # 16 sequences x 8 KV heads: 256 workgroups, no tail workgroup
    assert got[(2048, 10, 64)] == (4, 0)                                        # 8 sequences: 256 workgroups
    assert sum(got[(2048, 10, 32)]) * 32 <= 256 and sum(got[(8192, 10, 32)]) * 32 <= 256    # 4 sequences: at most 256 workgroups
    assert got[(2048, 10, 16)][0] == 16 and got[(2048, 10, 24)][0] == 16        # 2 and 3 sequences: one tile per wavefront
    assert sum(got[(4096, 10, 16)]) * 16 <= 256                                 # 2 sequences, K = 4096: no CU with two workgroups


def test_headline_shapes(table):
    merged = {(int(v[0]), int(v[1]), int(v[2])): (int(v[3]), int(v[4])) for kind, *v in table if kind == "merged"}
    assert merged[(2048, 10, 8)] == (16, 16)            # cfg2's partial step: 16 workgroups + the tail's own
    assert merged[(4096, 10, 4)][1] == 32               # cfg3 (4 KV heads, 7 heads per group: ticketed)
    assert merged[(8192, 10, 8)][1] == 32               # cfg5: ticketed with 32 workgroups
    emit = {(int(v[0]), int(v[1]), int(v[2])): int(v[3]) for kind, *v in table if kind == "emit"}
    assert emit[(33008, 1, 8)] * 8 == 512               # cfg2's full-cache kernel: 512 workgroups
    assert emit[(65536, 1, 4)] * 4 == 512               # cfg3
    assert emit[(131072, 1, 8)] * 8 == 1024             # cfg5
    for (length, b, hkv), n in emit.items():
        assert 1 <= n <= 1024 and n <= max((length + 127) // 128, 1)


def test_test_step_in_one_launch_is_resident_as_a_whole(table):
    """Both branches in one launch: one sequence, and the workgroups of either branch are all resident at once."""
    got = {}
    for kind, *v in table:
        if kind != "test_step":
            continue
        n, k, recent, batch, hkv, G, waves, nch, tail, inside, tiles = map(int, v)
        got[(n, k, recent, batch, hkv, G)] = tiles
        assert (waves != 0) == (tiles != 0)
        if waves:
            assert waves == 4 and tiles in (1, 2) and batch == 1 and inside >= 1
            assert max(nch + tail, inside) * hkv <= 512 and nch * 64 * tiles >= k and tail * 64 * tiles >= recent and nch <= 64 and nch + tail <= 65
    assert got[(66000, 4096, 1, 1, 4, 7)] == 1 and got[(33000, 2048, 64, 1, 8, 4)] == 1
    assert got[(66000, 4096, 65, 1, 4, 7)] == 2 and got[(33000, 4096, 1, 1, 8, 4)] == 2          # a 66th partial result; more than one workgroup per unit
    assert got[(33000, 8192, 1, 1, 8, 4)] == 0 and got[(33000, 2048, 1, 2, 8, 4)] == 0


def test_sliced_split_bounds_and_measured_choices(table):
    """Sizing of the partial step for the merge by slices: within what the merge takes and what is resident at once,
    never more workgroups than stretches of 128 rows, and the choices the measurements led to."""
    got = {}
    for kind, *v in table:
        if kind != "sliced":
            continue
        rows, tail, problems, n, own = map(int, v)
        got[(rows, tail, problems)] = (n, own)
        assert own in (0, 1) and 1 <= n and n + own <= 64
        assert (n + own) * problems <= 512
        counted = rows if tail <= 128 else rows + tail
        assert n <= max((counted + 127) // 128, 1)
        if tail > 128:
            assert own == 0
    assert len(got) == 12 * 3 * 4
    assert got[(2048, 10, 8)] == (16, 1)          # 16 workgroups of one tile per wavefront and the tail's own
    assert got[(4096, 10, 8)] == (32, 0)          # 32 x 8 = 256 workgroups: the tail's would be the only ones beyond one per CU
    assert got[(4096, 10, 4)] == (32, 1)
    assert got[(8192, 10, 8)] == (64, 0)          # a 65th partial result would cost every wavefront a second tile
    assert got[(8192, 10, 4)] == (64, 0)
    assert got[(16384, 10, 8)] == (64, 0)         # two tiles per wavefront either way
    assert got[(3072, 10, 8)] == (24, 1)


def test_partial_tile_form_bounds_and_measured_choices(table):
    """Every row has a wavefront's 16-row slot, the partial results have slots, and the launch is resident as a whole."""
    got, triggered = {}, {}
    for kind, *v in table:
        if kind != "tile":
            continue
        rows, pairs, tail, G, trig, waves, nch, ntail, exact = map(int, v)
        (triggered if trig else got)[(rows, pairs, tail, G)] = (waves, nch, ntail)
        assert waves in (0, 4, 8)
        if waves:
            assert nch * 16 * waves >= rows and ntail * 16 * waves >= tail and nch <= 64 and 1 <= nch + ntail <= (64 if exact else 65)
            assert (nch + ntail) * pairs <= (512 if waves == 4 else (256 if G > 4 else 512) if trig else 512 if G > 4 else 768)
            assert exact == (G > 4 and pairs > 16) and not (exact and G == 8 and nch + ntail <= (2 if waves == 4 else 3))
    assert got[(2048, 8, 1, 4)] == (4, 32, 1) and got[(256, 8, 1, 4)] == (4, 4, 1) and got[(4096, 4, 1, 8)] == (4, 64, 1)
    assert got[(4096, 8, 1, 4)] == (8, 32, 1) and got[(8192, 4, 1, 8)] == (8, 64, 1)
    assert got[(8192, 8, 1, 4)][0] == 0 and got[(1024, 128, 1, 4)][0] == 0            # 33 MB and more in many partial results
    assert got[(2048, 32, 1, 4)] == (8, 16, 1) and got[(1024, 64, 1, 4)] == (8, 8, 1) and got[(1024, 64, 1, 5)][0] == 0
    # the forms that the triggered cases of test_gpu_kernel_edges.py mean to reach
    assert triggered[(2048, 8, 1, 4)] == (4, 32, 1) and triggered[(700, 12, 1, 8)] == (4, 11, 1) and triggered[(700, 32, 1, 8)] == (8, 6, 1)
    assert triggered[(1024, 32, 1, 4)] == (8, 8, 1) and triggered[(2048, 32, 1, 4)][0] == 0 and triggered[(8192, 8, 1, 4)][0] == 0
    assert triggered[(1024, 32, 1, 8)][0] == 0 and triggered[(4096, 8, 1, 8)][0] == 0
    assert got[(0, 8, 500, 4)] == (4, 0, 8) and got[(2048, 8, 100000, 4)][0] == 0


def test_two_tile_form_bounds_and_measured_choices(table):
    """Every row has a slot (those since behind the small cache's where they have no workgroup), the partial results have theirs, the launch is
    resident as a whole."""
    got = {}
    for kind, *v in table:
        if kind != "two":
            continue
        rows, pairs, tail, G, fixed, waves, nch, ntail, exact, tiles, late = map(int, v)
        got[(rows, pairs, tail, G, fixed)] = (nch, ntail, late)
        if waves:
            assert (waves, tiles) == (8, 2) and exact == (G > 4 and pairs > 16)
            assert nch * 256 >= rows and 1 <= nch <= 64 and nch + ntail <= (64 if exact else 65) and (nch + ntail) * pairs <= 512
            assert ntail * 256 >= tail or (ntail == 0 and nch * 256 >= (max(rows, tail) if fixed else rows + tail))
            assert late == ((nch + ntail) * pairs > 256 or nch <= 3 or (ntail == 0 and tail > 256))      # (two per unit are bound by memory)
    assert got[(8192, 8, 11, 4, 1)] == (32, 0, 0) and got[(8192, 8, 11, 4, 0)] == (0, 0, 0)
    assert got[(8150, 8, 11, 4, 0)] == (32, 0, 0) and got[(6000, 8, 11, 4, 0)] == (24, 1, 0)
    assert got[(2000, 32, 11, 4, 0)] == (8, 0, 0) and got[(1000, 128, 11, 4, 0)] == (4, 0, 1) and got[(3000, 8, 11, 4, 0)] == (0, 0, 0)
    assert got[(1700, 64, 11, 4, 0)] == (7, 0, 1) and got[(500, 128, 11, 4, 0)] == (2, 0, 1) and got[(1000, 64, 257, 4, 1)] == (4, 0, 1)
    # no gain, or less than short rows lose: one workgroup to a pair, 16 pairs at two per unit, few to a pair of groups of 8
    assert got[(256, 128, 1, 4, 1)] == (0, 0, 0) and got[(8150, 16, 11, 4, 0)] == (0, 0, 0) and got[(1000, 128, 11, 8, 0)] == (0, 0, 0)


def test_selection_parts_are_resident_at_once(table):
    got = {int(v[0]): int(v[1]) for kind, *v in table if kind == "parts"}
    for rows, parts in got.items():
        assert parts in (1, 2, 4, 8) and (parts == 1 or rows * parts <= 256) and (parts == 8 or rows * parts > 128), (rows, parts)


def test_few_long_rows_are_listed(table):
    """... where that was measured to be faster; wherever it is, the workspace has room for the list, and what is sized for
    longer rows or more ranks serves shorter ones and fewer."""
    got = {tuple(map(int, v[:3])): tuple(map(int, v[3:])) for kind, *v in table if kind == "listed"}
    assert len(got) == 8 * 7 * 8
    for (n, k, rows), (listed, room, grows) in got.items():
        assert grows and (room or not listed) and (not room or rows <= 6), (n, k, rows)
        few = k <= 4096 or (rows <= 3 and k <= 8192)
        assert listed == (rows <= (6 if k <= 4096 else 4) and n >= 49152 and n >= (16 if few else 20) * k), (n, k, rows)


def test_selection_stretches_leave_no_rank_out(table):
    """Every part's stretch ends where the next one's starts, and the last part looks at its bin down to the floor wherever its
    estimate leaves it nothing (bins of tens of millions of positions, few ranks): no rank stays unwritten."""
    seen = {(int(v[0]), int(v[1])): tuple(map(int, v[2:])) for kind, *v in table if kind == "stretch"}
    assert len(seen) == 42
    for key, (unwritten, order, empty) in seen.items():
        assert unwritten == 0 and order == 0, key
    assert seen[(1 << 28, 3)][2] > 100 and seen[(40000000, 3)][2] > 0 and seen[(20000000, 3)][2] == 0      # the case does come up


@pytest.fixture(scope="module")
def inside(table):
    got = {tuple(map(int, v[:4])): tuple(map(int, v[4:])) for kind, *v in table if kind == "inside"}
    assert len(got) == 14 * 9 * 8 * 3
    return got


def test_inside_split_bounds(inside):
    """Full passes merged inside the kernel: within the slots of the merge and the stretches of 128 rows; the pooling
    kernels of a deferred step are told the number that was launched."""
    for (rows, b, hkv, G), (n, emit, deferred, fp32) in inside.items():
        assert 0 <= n <= 64 and n <= max((rows + 127) // 128, 1)
        assert deferred == (n if n > 0 else emit) and deferred >= 1
        if fp32:
            assert n == emit and G <= 4 and (b == 1 or b > 64) and n * b * hkv <= 512
        if G > 4:
            assert n <= 1 or n * b * hkv <= 512


def test_inside_split_is_not_given_up_for_a_remainder(inside):
    """A number of (sequence, KV head) pairs that does not divide 256 leaves a few workgroups fewer whichever launch merges."""
    for key, n in {(16384, 1, 5, 4): 51, (20000, 1, 6, 4): 42, (6000, 6, 4, 4): 10, (8000, 3, 8, 1): 10}.items():
        assert inside[key][0] == n == inside[key][1], key
    for (rows, b, hkv, G), (n, emit, _, _) in inside.items():
        if n == 0 and (hkv > 2 or b == 1 or b > 64 or rows <= 8192):
            assert min(emit, 64) * b * hkv < 256 and (min(emit, 64) + 1) * b * hkv <= 256, (rows, b, hkv, G)


def test_inside_split_leaves_no_part_of_a_round(inside):
    """Where the slots of the merge bind, the total is as near below a multiple of the 256 compute units as the pairs allow."""
    for key, n in {(131072, 3, 4, 4): 42, (131072, 3, 3, 4): 56, (131072, 1, 5, 4): 51, (131072, 1, 7, 4): 36, (131072, 1, 6, 7): 42,
                   (131072, 1, 4, 7): 64, (131072, 1, 8, 4): 64, (65536, 2, 8, 4): 32, (131072, 65, 1, 4): 15}.items():
        assert inside[key][0] == n, key
    for (rows, b, hkv, G), (n, emit, _, _) in inside.items():
        total = n * b * hkv
        if total > 256 and n == 64:
            assert total == 512, (rows, b, hkv, G)
        if 0 < n < 64 and n < emit and G <= 4 and rows > 8192:       # trimmed: one workgroup more per pair would be the remainder
            assert total <= 512 and (total + b * hkv > 512 or 256 - b * hkv < total <= 256), (rows, b, hkv, G)


def test_one_long_sequence_of_a_ragged_batch_can_fill_the_chip(inside):
    """With one or two KV heads the 64 slots of the merge inside would hold a long sequence to 64 or 128 workgroups: the
    launch with up to 256 partial results to a sequence and KV head, and the merge launch, instead."""
    for (rows, b, hkv, G), (n, emit, deferred, _) in inside.items():
        if 1 < b <= 64 and hkv <= 2 and rows > 8192:
            assert n == 0 and deferred == emit, (rows, b, hkv, G)
        if 1 < b <= 64 and hkv > 2 and rows * b >= 65536:
            assert n > 0, (rows, b, hkv, G)


def test_window_form_bounds_and_measured_choices(table):
    got = {}
    for kind, *v in table:
        if kind != "window":
            continue
        rows, pairs, blocks, limit, T, wg_rows, nch = map(int, v)
        got[(rows, pairs, blocks)] = (T, nch)
        assert 1 <= nch <= limit and nch <= max((rows + wg_rows - 1) // wg_rows, 1)
        assert (T, wg_rows) in ((1, 128), (2, 128), (4, 512))
        if T != 2:
            assert nch == 1 or nch * pairs <= 512
    assert got[(32768, 8, 8)] == (4, 64)          # 32 queries of 4 heads: every wavefront of the chip 64 rows
    assert got[(32768, 8, 1)][0] == 2             # one query
    assert got[(2100, 8, 8)][0] == 1 and got[(40000, 1, 8)][0] == 1
    assert got[(1100, 260, 2)] == (2, 2) and got[(513, 128, 16)] == (4, 2)
    # a last round of T = 4 with little in it (with 4 KV heads it takes 65536 rows to a round, with 8 32768)
    assert got[(1400, 260, 3)] == (4, 1) and got[(1100, 260, 3)][0] == 2
    assert got[(36000, 8, 3)][0] == 2 and got[(36000, 8, 8)][0] == 2 and got[(36000, 8, 16)][0] == 4
    assert got[(76000, 4, 3)][0] == 2 and got[(64000, 8, 3)][0] == 4 and got[(64000, 8, 8)][0] == 4
    assert got[(16000, 8, 3)][0] == 2 and got[(16000, 8, 8)][0] == 4          # half a round: fewer workgroups, none of them idle


def test_h2o_split_bounds(table):
    seen = 0
    for kind, *v in table:
        if kind != "h2o":
            continue
        rows, b, hkv, n, emit, slots = map(int, v)
        assert 1 <= n <= slots                    # partial results the workspace of budget + 1 rows has room for
        tiles = (rows + 31) // 32 * b * hkv
        if not 10240 <= tiles < 14336:            # 768 workgroups are a choice here only
            assert n == emit, (rows, b, hkv)
        seen += 1
    assert seen == 9 * 4 * 3


# What the lists of test_gpu_kernel_edges.py mean to reach: (wavefronts, tiles to each, workgroups of the small cache and of the rows since, (max, sum)
# pairs, late), no wavefronts: attn_split_kernel; the trigger's without tiles and late; (tiles, workgroups) of the test steps in one launch; (wavefronts,
# workgroups, pairs) of the gather inside the step, no wavefronts: two launches.
FORMS = {
    "tile": {
        "k1": (4, 1, 1, 1, 0, 0), "k16_17_g1": (4, 1, 1, 1, 0, 0), "k63_g8": (4, 1, 1, 2, 0, 0), "k64_g5": (4, 1, 1, 1, 0, 0),
        "k65_evict": (4, 1, 2, 1, 0, 0), "k256_evicts_all": (4, 1, 4, 5, 0, 0), "none_selected": (4, 1, 0, 4, 0, 0),
        "k1280_20_chunks": (4, 1, 20, 1, 0, 0), "k2560_g7": (4, 1, 40, 1, 0, 0), "k2561_u4": (4, 1, 41, 1, 0, 0),
        "k4096_65_chunks_g7": (4, 1, 64, 1, 0, 0), "k4096_8w": (8, 1, 32, 1, 0, 0), "two_17_g6": (8, 2, 17, 1, 0, 0),
        "two_32_g8": (8, 2, 32, 1, 0, 0), "k7900_63_chunks_8w_g7": (8, 1, 62, 1, 0, 0), "k3900_8w_g8": (8, 1, 31, 1, 0, 0),
        "k8192_split": (0, 0, 0, 0, 0, 0), "batch": (8, 1, 6, 1, 0, 0), "batch_3_per_cu": (8, 1, 4, 1, 0, 0), "exact_g7": (4, 1, 5, 1, 1, 0),
        "exact_g8_8w": (8, 1, 4, 1, 1, 0), "two_exact_g5_11": (8, 2, 11, 1, 1, 0), "exact_g5_25_chunks": (8, 1, 24, 1, 1, 0),
        "exact_g6_empty": (4, 1, 2, 2, 1, 0), "two_own_tail": (8, 2, 24, 1, 0, 0), "two_inside_8150": (8, 2, 32, 0, 0, 0),
        "two_inside_fixed": (8, 2, 32, 0, 0, 1), "two_inside_fixed_17": (8, 2, 32, 0, 0, 0), "two_inside_fixed_256": (8, 2, 32, 0, 0, 0),
        "two_batch": (8, 2, 8, 0, 0, 0), "two_batch_fixed": (8, 2, 8, 0, 0, 0), "two_512": (8, 2, 7, 0, 0, 1),
        "two_g7_64_results": (8, 2, 63, 1, 0, 0), "two_exact_g8": (8, 2, 8, 0, 1, 0), "two_exact_g5_fixed": (8, 2, 6, 0, 1, 0),
        "two_g1": (8, 2, 16, 0, 0, 0), "late_halves": (8, 2, 7, 0, 0, 1), "late_2_of_440": (8, 2, 2, 0, 0, 1), "late_fixed_300": (8, 2, 4, 0, 0, 1),
        "late_exact_g5_24_results": (8, 2, 24, 0, 1, 1), "late_exact_g7_own_tail": (8, 2, 23, 1, 1, 1), "late_g8_15": (8, 2, 15, 0, 1, 1)},
    "triggered": {
        "tile_4w": (4, 32, 1, 0), "tile_4w_g8": (4, 11, 1, 0), "tile_8w": (8, 8, 1, 0), "tile_8w_g7": (8, 9, 1, 0), "tile_8w_exact_g8": (8, 6, 1, 1),
        "split_tagged_long": (0, 0, 0, 0), "split_tagged_batch": (0, 0, 0, 0), "split_tagged_g8": (0, 0, 0, 0), "split_ticketed_g7": (0, 0, 0, 0)},
    "test_step": [
        (1, 32, 1), (1, 32, 1), (1, 64, 1), (1, 11, 1), (1, 2, 1), (1, 4, 1), (1, 1, 1), (1, 1, 1), (1, 8, 1), (1, 16, 1), (1, 1, 1), (1, 32, 3),
        (2, 32, 1), (2, 32, 2), (2, 24, 1), (2, 32, 1), (2, 63, 1)],
    "gather": [
        (8, 64, 0), (4, 32, 0), (4, 2, 0), (8, 33, 0), (4, 1, 0), (4, 2, 0), (4, 4, 0), (8, 9, 0), (4, 8, 1), (4, 5, 1), (0, 0, 0), (0, 0, 0),
        (8, 8, 1)]}


def test_edge_cases_reach_the_forms_they_are_for(tmp_path):
    import test_gpu_kernel_edges as edges
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    body = []
    for name, G, Hkv, k, recent, evict, seqs in edges.TILE_EDGES:
        pairs = len(seqs) * Hkv
        body.append("f = two_tile_form(%d, %d, %d, %d, %d); if (f.waves == 0) f = partial_tile_form(%d, %d, %d, %d, false);" % (k, recent, pairs, G, evict, k, recent, pairs, G))
        body.append('printf("%d %d %d %d %d %d\\n", f.waves, f.tiles, f.nch, f.tail, (int)f.exact, (int)f.late);')
    for G, Hkv, B, k, recent, fixed in edges.TRIGGERED.values():
        body.append("f = partial_tile_form(%d, %d, %d, %d, true);" % (k, recent, B * Hkv, G))
        body.append('printf("%d %d %d %d\\n", f.waves, f.nch, f.tail, (int)f.exact);')
    for G, Hkv, n, k, recent, fixed in edges.TEST_STEPS:
        body.append("{ rk_geom g{1, %d, %d, 128, 1.f}; f = test_step_form(&g, %d, %d, %d); }" % (G * Hkv, Hkv, k, max(recent, 1), n))
        body.append('printf("%d %d %d\\n", f.tiles, f.nch, f.tail);')
    for G, Hkv, B, n, k in edges.GATHER_ATTN:
        body.append("f = partial_tile_form(%d, 0, %d, %d, false);" % (k, B * Hkv, G))
        body.append('printf("%d %d %d\\n", f.waves, f.nch, (int)f.exact);')
    src, exe = tmp_path / "forms.cpp", tmp_path / "forms"
    src.write_text('#include "rk_internal.h"\n#include <cstdio>\nusing namespace rk;\nint main() {\n    TileForm f;\n%s\n    return 0;\n}\n' % "\n".join(body))
    r = subprocess.run([hipcc, "-O1", "-std=c++17", "-I", CSRC, "-x", "hip", "--offload-arch=gfx950", str(src), "-o", str(exe)],
                       capture_output=True, text=True, timeout=600)
    assert r.returncode == 0, r.stderr[-2000:]
    got = [tuple(map(int, ln.split())) for ln in subprocess.run([str(exe)], capture_output=True, text=True, timeout=60).stdout.splitlines()]
    assert list(FORMS["tile"]) == [c[0] for c in edges.TILE_EDGES] and list(FORMS["triggered"]) == list(edges.TRIGGERED)
    names = [*FORMS["tile"], *FORMS["triggered"], *edges.TEST_STEPS, *edges.GATHER_ATTN]
    want = [*FORMS["tile"].values(), *FORMS["triggered"].values(), *FORMS["test_step"], *FORMS["gather"]]
    assert len(got) == len(want) == len(names)
    assert [(n, g) for n, g, w in zip(names, got, want) if g != w] == []
