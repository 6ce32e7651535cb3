"""Sizes at which a kernel's tiles, rounds and dispatch rules change hands, against the CPU oracle."""
import ctypes
import sys

import numpy as np
import pytest
import torch

import gen
import oracle
from helpers import assert_idx_equivalent

pytestmark = pytest.mark.gpu

SCALE = float(np.float32(1 / np.sqrt(128)))


@pytest.fixture(scope="module")
def rk():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_05787_amd as lib
    return lib


def say(*a):
    print(*a, file=sys.stderr, flush=True)


def draw(seed, *shape):
    return torch.randn(*shape, generator=torch.Generator().manual_seed(seed)).to(torch.bfloat16)


# Up to 65536 rows over all pairs 16 rows per wavefront, 128 per workgroup; beyond, two sets of 32 rows and 128 per workgroup
# for up to 32 columns ("narrow", 520 and 260 pairs: one and two workgroups to a pair) and where rounds of 512 rows per
# workgroup would be left half empty ("half_empty"), 64 rows and 512 per workgroup for the rest ("wide" and the last but one: one
# workgroup to a pair, and four).  Lengths around whole tiles and steps, in either of the
# two sets, and, less the window, around the first row that not every query sees; groups with columns that do not exist (3, 5
# and 7 heads), blocks of columns that the queries do not fill, 16 blocks, and a negative scale.
WINDOW_EDGES = [("rows_63_64_65", 3, 8, 2, [63, 64, 65], 5, SCALE), ("rows_511_512_513", 3, 4, 4, [511, 512, 513], 32, SCALE),
                ("rows_575_576_577_w1", 3, 8, 1, [575, 576, 577], 1, SCALE), ("narrow_1100r", 65, 8, 8, [1100, 1025] + [40] * 63, 3, SCALE),
                ("narrow_g3_sets", 65, 12, 4, [130, 300, 1090] + [40] * 62, 3, SCALE),
                ("wide_g3_w12", 65, 12, 4, [1036, 1035, 1400] + [40] * 62, 12, SCALE), ("wide_g7_w5", 65, 28, 4, [1025, 1024, 1400] + [40] * 62, 5, SCALE),
                ("wide_g5_w9", 65, 20, 4, [513, 512, 1000] + [65] * 62, 9, SCALE), ("half_empty_g7", 65, 28, 4, [1025, 1055, 1093] + [40] * 62, 5, SCALE),
                ("half_empty_g5", 65, 20, 4, [511, 600, 512] + [65] * 62, 14, SCALE),
                ("g8_w32_two_rounds", 128, 8, 1, [2100, 2049] + [33] * 126, 32, SCALE), ("negative_scale", 1, 8, 2, [700], 9, -SCALE)]


@pytest.mark.parametrize("case", WINDOW_EDGES, ids=[c[0] for c in WINDOW_EDGES])
def test_window_select_at_tile_edges(rk, case):
    """Votes to 1e-5 relative (fp32 scores of magnitude up to ~10: 2^-24 x 10 in the exponent, twice), the selection
    to the oracle's score gaps; sequences beyond the first three are padding and only checked for being finite."""
    name, B, Hq, Hkv, lens, W, scale = case
    say("window edge", name)
    cap, k = max(lens) + 3, 48
    K, qw = draw(len(name), B, Hkv, cap, 128), draw(len(name) + 1, B, W, Hq, 128)
    for b in range(B):
        K[b, :, lens[b]:] = float("nan")                 # rows past the end must not matter
    geom = rk.Geom(B, Hq, Hkv, 128, scale)
    ws = rk.Workspace(geom, cap, k)
    votes = torch.full((B, Hq, cap), -7.0, device="cuda")
    idx = torch.full((B, Hkv, k), -5, dtype=torch.int32, device="cuda")
    rk.rk_window_select(geom, qw.cuda(), K.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda"), max(lens), k, 7,
                        idx, votes=votes, workspace=ws)
    torch.cuda.synchronize()
    assert torch.isfinite(votes).all()
    n_ref, G = min(B, 3), Hq // Hkv
    v_ref = oracle.window_votes(gen.bf16_bits(qw[:n_ref]), gen.bf16_bits(K[:n_ref]), lens[:n_ref], scale)
    i_ref, _ = oracle.topk_select(v_ref.astype(np.float32), lens[:n_ref], Hkv, k, 7)
    for b in range(n_ref):
        n, vn = lens[b], votes[b].cpu().numpy()
        assert (np.abs(vn[:, :n] - v_ref[b, :, :n]) / v_ref[b, :, :n]).max() < 1e-5
        assert (vn[:, n:] == -7.0).all()
        for g in range(Hkv):
            P = oracle.pooled_group_scores(v_ref[b, g * G:(g + 1) * G, :n].astype(np.float32), 7)
            assert_idx_equivalent(idx[b, g].cpu().numpy(), i_ref[b, g], P, n, k, "%s b=%d g=%d" % (name, b, g))


# The (max, sum) pairs of pass 1 folded in pass 2 (16 per thread: one workgroup's, 64 workgroups' of 128 columns, 256 workgroups'
# of 16) and by the launch between the passes (65 workgroups, 80 columns).
WINDOW_FOLDS = [("one_row", 1, 8, 2, [1], 3, SCALE), ("128_columns_64_wgs", 1, 4, 1, [8192], 32, SCALE), ("128_columns_65_wgs", 1, 4, 1, [8193], 32, SCALE),
                ("16_columns", 2, 4, 1, [32768, 129], 4, SCALE), ("80_columns", 2, 8, 2, [3000, 60], 20, SCALE)]


@pytest.mark.parametrize("case", WINDOW_FOLDS, ids=[c[0] for c in WINDOW_FOLDS])
def test_window_select_folds_pass_1(rk, case):
    test_window_select_at_tile_edges(rk, case)


# (rows, queries, largest score of the unrelated rows, a row that one query is aligned with, sign of the scale)
WINDOW_SCORES = [(3000, 8, 5, True, 1), (3000, 8, 20, True, 1), (3000, 32, 100, True, 1), (40000, 32, 100, True, -1), (3000, 8, 400, False, 1),
                 (40000, 20, 400, True, 1), (9000, 3, 400, False, -1), (3000, 8, 1000, False, 1), (700, 5, 0, False, 1)]


@pytest.mark.parametrize("case", WINDOW_SCORES, ids=["n%d_w%d_s%d_%d_%d" % c for c in WINDOW_SCORES])
def test_window_votes_of_peaked_and_large_scores(rk, case):
    """Keys and queries of whole numbers, so that products are exact and what is seen is the softmax alone: votes of at least
    1e-3 of the largest one are off by the rounding of the scale and of one exponent of at most 7 log2 e = 10 (2 x 10 x 2^-24 x ln 2 = 8e-7),
    the exponential's last place and sums (a few 2^-24), whatever the size of the scores."""
    n, W, top, peak, sign = case
    say("window votes", *case)
    Hkv, G = 2, 4
    g = torch.Generator(device="cuda").manual_seed(n + W + top)
    whole = lambda *shape: torch.randint(-4, 5, shape, generator=g, device="cuda").to(torch.bfloat16)
    K, q = whole(1, Hkv, n, 128), whole(1, W, Hkv * G, 128)
    scale = sign * float(np.float32(top / 300.0))                    # products of unrelated rows reach about 300
    if peak:
        K[0, 1, n // 3] = sign * q[0, W - 1, G]
    geom = rk.Geom(1, Hkv * G, Hkv, 128, scale)
    ws = rk.Workspace(geom, n, 64)
    votes = torch.zeros(1, Hkv * G, n, device="cuda")
    idx = torch.empty(1, Hkv, 64, dtype=torch.int32, device="cuda")
    rk.rk_window_select(geom, q, K, torch.tensor([n], dtype=torch.int32, device="cuda"), n, 64, 1, idx, votes=votes, workspace=ws)
    torch.cuda.synchronize()
    x = torch.matmul(q[0].double().view(W, Hkv, G, 128).permute(1, 2, 0, 3).reshape(Hkv, G * W, 128), K[0].double().transpose(1, 2).contiguous())
    z = (scale * x).view(Hkv, G, W, n)
    for i in range(W):
        z[:, :, i, n - W + i + 1:] = -float("inf")
    ref = torch.softmax(z, -1).sum(2).reshape(Hkv * G, n)
    big = ref >= 1e-3 * ref.amax(1, keepdim=True)
    err = ((votes[0].double() - ref).abs() / ref)[big].max().item()
    print("largest relative error %.3g" % err, file=sys.stderr, flush=True)
    assert err <= 2e-6


@pytest.mark.parametrize("shape", [(4, 1, 2, 700), (1, 3, 2, 700), (4, 5, 8, 9000), (4, 13, 8, 9000), (4, 13, 8, 32000), (2, 1, 8, 33000), (3, 7, 8, 33000)],
                         ids=lambda s: "g%d_w%d_h%d_n%d" % s)
def test_window_select_with_infinite_keys(rk, shape):
    """A key with an infinite component and minus infinity as every query's score gets no vote, as one does whose scores are
    finite and hopeless: the same votes, bit for bit, and the same selection (a window that does not fill its last block of
    16 columns; few rows, few columns, and 64 rows per wavefront)."""
    G, W, Hkv, n = shape
    say("window with infinite keys", shape)
    k, Hq = 64, G * Hkv
    q, K = draw(n + W, 1, W, Hq, 128), draw(n + G, 1, Hkv, n, 128)
    q[..., 5] = -1.0
    rows = torch.tensor([0, 17, n // 2, n - W - 130])
    geom = rk.Geom(1, Hq, Hkv, 128, SCALE)
    got = []
    for hopeless in (1e30, float("inf")):
        K[:, :, rows, 5] = hopeless
        ws = rk.Workspace(geom, n, k)
        votes = torch.zeros(1, Hq, n, device="cuda")
        idx = torch.full((1, Hkv, k), -5, dtype=torch.int32, device="cuda")
        rk.rk_window_select(geom, q.cuda(), K.cuda(), torch.tensor([n], dtype=torch.int32, device="cuda"), n, k, 1, idx,
                            votes=votes, workspace=ws)
        torch.cuda.synchronize()
        got.append((votes.cpu(), idx.cpu()))
    assert (got[1][0][:, :, rows] == 0).all()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


# (group, pooling width, rows): the tiles of the pooling kernels end at multiples of 512, 1024 (from 98304 rows on) and,
# batched over layers, 2048
POOL_EDGES = [(4, 7, 512), (4, 7, 513), (1, 7, 1021), (7, 7, 1023), (8, 7, 1030), (4, 1, 700), (5, 15, 1537), (2, 63, 515),
              (4, 7, 2047), (4, 7, 2051), (3, 7, 3), (4, 7, 1), (4, 7, 98309)]


@pytest.mark.parametrize("spread", ["plain", "near_ties", "far_apart"])
@pytest.mark.parametrize("shape", POOL_EDGES, ids=["g%d_w%d_n%d" % s for s in POOL_EDGES])
def test_group_maximum_by_one_exponential_is_exact(rk, shape, spread):
    """The selection without returned weights (one exponential per position, of the head with the largest exponent)
    against the same call with them (all heads' weights, their maximum): the same positions and the same scores
    bit for bit, also batched over two layers.  near_ties: heads that are copies of one another, or differ in
    the last bit of a few dimensions; far_apart: scores of magnitude 100 and more, weights down to subnormal and zero."""
    G, pool_w, n = shape
    say("one exponential", shape, spread)
    B, Hkv, k = (1, 1, 64) if n > 50000 else (2, 2, 40)
    Hq, cap = G * Hkv, n + 5
    q, K, V = draw(G + n, B, Hq, 128), draw(n, B, Hkv, cap, 128), draw(n + 1, B, Hkv, cap, 128)
    if spread == "near_ties":
        q = q.view(B, Hkv, G, 128)
        q[:, :, 1:] = q[:, :, :1]                        # every head of a group equal to the first ...
        bits = q.view(torch.int16)
        bits[:, :, G // 2:, ::40] ^= 1                   # ... or one unit in the last place away in four dimensions
        q = q.view(B, Hq, 128)
    elif spread == "far_apart":
        q = (q.float() * 30).to(torch.bfloat16)
    lens = [n] * B if B == 1 else [n, max(n - 3, 0)]
    geom = rk.Geom(B, Hq, Hkv, 128, SCALE)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    q, K, V = q.cuda(), K.cuda(), V.cuda()
    got = []
    for want in (False, True):
        ws = rk.Workspace(geom, cap, k)
        out = torch.zeros(B, Hq, 128, dtype=torch.bfloat16, device="cuda")
        idx = torch.full((B, Hkv, k), -5, dtype=torch.int32, device="cuda")
        sel = torch.full((B, Hkv, k), -5.0, device="cuda")
        w = torch.zeros(B, Hq, cap, device="cuda") if want else None
        rk.rk_full_attn_select(geom, q, K, V, sl, n, out, k, pool_w, idx, weights=w, sel_scores=sel, workspace=ws)
        got.append((idx.cpu(), sel.cpu(), out.cpu()))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    # ... and what the maximum over the returned weights selects
    A = w.view(B, Hkv, G, cap).amax(2).cpu().numpy()
    for b in range(B):
        for g in range(Hkv):
            P = oracle.pooled_group_scores(A[b, g, None, :lens[b]], pool_w)
            order = np.lexsort((np.arange(lens[b]), -P))[:k]
            assert (got[0][0][b, g, :len(order)].numpy() == order).all()
            assert (got[0][1][b, g, :len(order)].numpy() == P[order].astype(np.float32)).all()
    wss = [rk.Workspace(geom, cap, k) for _ in range(2)]
    small = torch.zeros(2, 2, B, Hkv, k, 128, dtype=torch.bfloat16, device="cuda")
    idx = torch.full((2, B, Hkv, k), -5, dtype=torch.int32, device="cuda")
    tail = torch.zeros(2, B, dtype=torch.int32, device="cuda")
    layers = (type(rk.layer_state(geom, K, V, small[0, 0], small[0, 1], idx[0], tail[0], k=k)) * 2)(
        *[rk.layer_state(geom, K, V, small[l, 0], small[l, 1], idx[l], tail[l], k=k) for l in range(2)])
    for l in range(2):
        rk.rk_full_attn_deferred(geom, q, K, V, sl, n, out, workspace=wss[l])
    import ctypes
    rk.rk_refresh_batched(geom, layers, (ctypes.c_void_p * 2)(*[x.ptr for x in wss]), wss[0].nbytes, sl, n, k, pool_w=pool_w)
    torch.cuda.synchronize()
    for l in range(2):
        assert torch.equal(idx[l].cpu(), got[0][0])


# the workgroups of a launch over 2..64 sequences are shared out by length, with exact remainders
RAGGED = [("two_far_apart", [9000, 1]), ("three_equal", [1280, 1280, 1280]), ("ties", [300, 300, 301, 0, 299, 300]),
          ("one_long_of_64", [30000] + [1, 0, 129] * 21), ("steps_64", [128 * i for i in range(64)]), ("beyond_64", [200] * 64 + [4000]),
          ("one_short", [700]), ("one_of_8192", [8192]), ("one_of_8193", [8193]), ("four_of_9000", [9000, 8999, 8193, 9000]),
          ("primes", [7919, 6007, 4999, 3001, 2003, 1009, 503, 251, 127, 61, 31])]


@pytest.mark.parametrize("G", [1, 4, 7])
@pytest.mark.parametrize("case", RAGGED, ids=[c[0] for c in RAGGED])
def test_ragged_batches_cover_every_row_once(rk, case, G):
    """Full attention over batches of very different lengths, with weights, without, and deferred, against fp64: a row
    left out or taken twice by the shares would move lse by far more than its bound (1e-5)."""
    name, lens = case
    say("ragged", name, G)
    B, Hkv, cap = len(lens), 2, max(lens) + 2
    g = torch.Generator(device="cuda").manual_seed(B + G)
    K = torch.randn(B, Hkv, cap, 128, generator=g, device="cuda").to(torch.bfloat16)
    V = torch.randn(B, Hkv, cap, 128, generator=g, device="cuda").to(torch.bfloat16)
    q = torch.randn(B, Hkv * G, 128, generator=g, device="cuda").to(torch.bfloat16)
    geom = rk.Geom(B, Hkv * G, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, cap, 16)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    runs = []
    for kind in ("weights", "plain", "deferred"):
        out = torch.full_like(q, 7.0)
        lse = torch.full((B, Hkv * G), 7.0, device="cuda")
        if kind == "deferred":
            rk.rk_full_attn_deferred(geom, q, K, V, sl, max(lens), out, lse=lse, workspace=ws)
        else:
            w = torch.zeros(B, Hkv * G, cap, device="cuda") if kind == "weights" else None
            rk.rk_full_attn(geom, q, K, V, sl, max(lens), out, weights=w, lse=lse, workspace=ws)
        runs.append((kind, out, lse))
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        if n == 0:
            for kind, out, lse in runs:
                assert (out[b] == 0).all() and (lse[b] == -float("inf")).all(), (name, kind, b)
            continue
        s = SCALE * torch.matmul(q[b].double().view(Hkv, G, 128), K[b, :, :n].double().transpose(1, 2).contiguous())
        z = torch.logsumexp(s, dim=-1)
        ref = torch.matmul(torch.exp(s - z[..., None]), V[b, :, :n].double()).reshape(-1, 128)
        for kind, out, lse in runs:
            assert (lse[b].double() - z.reshape(-1)).abs().max() < 1e-5, (name, kind, b)
            d = (out[b].double() - ref).abs()             # one bf16 step of the larger value, and 4e-6 (see helpers)
            assert (d <= torch.maximum(out[b].double().abs(), ref.abs()) * 2.0 ** -7 + 4e-6).all(), (name, kind, b)


@pytest.mark.parametrize("G", [1, 4, 5, 6, 7, 8])
@pytest.mark.parametrize("case", [("slices_64", 4, [8192]), ("slices_64_long", 4, [33000]), ("longer", 4, [90000]), ("ragged", 4, [5000, 9000, 4097, 8192]),
                                  ("last_arrival", 4, [16500] * 10), ("slices_21", 8, [9000] * 3), ("one_long", 4, [30000] + [4100] * 7)],
                         ids=lambda c: c[0])
def test_output_merged_inside_is_normalised_in_fp64(rk, case, G):
    """Full passes that merge their partial results in the streaming kernel, at scores around 4096: a log-sum-exp of that
    size rounded to fp32 moves the weight of a whole partial result by up to 2.4e-4, an output of rows that cancel by
    about 2e-5.  The scores are exact here (whole multiples of 2^-6 below 2^13), so the bound is what is left: 2^-17 of
    P's two bf16 parts and 3e-7 of an exponential, on 4097 and more weights that add up to 1 and meet at random signs (below 1e-6), twice.
    The bits are those of the pass that returns its weights, whose merge is a launch of its own.  (8 heads: 21 partial
    results have no merge by slices, the last arrival takes them in two rounds.)"""
    name, Hkv, lens = case
    say("inside merge", name, G)
    B, cap = len(lens), max(lens)
    in_fp32 = B == 1 and G <= 4 and cap < 80000             # deferred: one residency round, merged like a partial step
    g = torch.Generator(device="cuda").manual_seed(B + 10 * G)
    q = torch.zeros(B, Hkv * G, 128, device="cuda")
    q[..., 0], q[..., 1] = 64.0, 1.0
    K = torch.zeros(B, Hkv, cap, 128, device="cuda")
    K[..., 0], K[..., 1] = 64.0, torch.randint(-128, 129, (B, Hkv, cap), generator=g, device="cuda") / 64.0
    sign = 1.0 - 2.0 * (torch.arange(cap, device="cuda") // 128 % 2)
    V = sign[:, None].expand(B, Hkv, cap, 128).contiguous()
    for b, n in enumerate(lens):                            # the last rows bring the output to nearly nothing
        w = torch.softmax(K[b, :, :n, 1].double(), dim=-1)
        for r in range(max(n - 4, 0), n):
            V[b, :, r] = 0
            V[b, :, r] = (-torch.matmul(w[:, None], V[b, :, :n].double())[:, 0] / w[:, r, None]).to(torch.bfloat16).float()
    q, K, V = q.to(torch.bfloat16), K.to(torch.bfloat16), V.to(torch.bfloat16)
    geom = rk.Geom(B, Hkv * G, Hkv, 128, 1.0)
    ws = rk.Workspace(geom, cap, 16)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    outs = []
    for kind in ("deferred", "plain", "weights"):
        out, lse = torch.full_like(q, 7.0), torch.full((B, Hkv * G), 7.0, device="cuda")
        if kind == "deferred":
            rk.rk_full_attn_deferred(geom, q, K, V, sl, cap, out, lse=lse, workspace=ws)
        else:
            w = torch.zeros(B, Hkv * G, cap, device="cuda") if kind == "weights" else None
            rk.rk_full_attn(geom, q, K, V, sl, cap, out, weights=w, lse=lse, workspace=ws)
        outs.append((kind, out, lse))
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        s = 4096.0 + K[b, :, :n, 1].double()
        z = torch.logsumexp(s, dim=-1)
        ref = torch.matmul(torch.exp(s - z[:, None])[:, None], V[b, :, :n].double())              # [Hkv, 1, 128]
        for kind, out, lse in outs:
            if kind == "plain" and not (B == 1 and cap > 8192):
                continue                                    # few rows to a pair: the merge of the partial steps
            if kind == "deferred" and in_fp32:
                continue
            assert (out[b].double().view(Hkv, G, 128) - ref).abs().max() < 2e-6, (name, kind, b)
            assert (lse[b].double().view(Hkv, G) - z[:, None]).abs().max() <= 4.9e-4, (name, kind, b)      # fp32 at 4096: 2^-11
    if B == 1 and cap > 8192 and cap < 80000:
        assert torch.equal(outs[1][1], outs[2][1]), name
    if not in_fp32 and name not in ("longer", "one_long") and (name != "last_arrival" or G <= 4):      # (the others are split otherwise)
        assert torch.equal(outs[0][1], outs[2][1]), name


@pytest.mark.parametrize("case", [(7, 4, [33000]), (4, 8, [9000, 8000, 8999]), (2, 4, [2000] * 16), (4, 4, [33000]), (8, 8, [9000] * 3), (3, 4, [700] * 30)],
                         ids=lambda c: "g%d_%d_pairs_n%d" % (c[0], c[1] * len(c[2]), c[2][0]))
def test_full_passes_hand_over_slices_to_the_last_workgroup(rk, case):
    """Full passes merged by slices with the bound on re-reads of rows in flight at 0 (every workgroup leaves its slice to
    the one that publishes last), 1, 2 and its default: the same bits, out and lse, call after call on one workspace."""
    G, Hkv, lens = case
    say("hand-over", case)
    B, cap = len(lens), max(lens)
    g = torch.Generator(device="cuda").manual_seed(G + cap)
    K, V = (torch.randn(B, Hkv, cap, 128, generator=g, device="cuda").to(torch.bfloat16) for _ in range(2))
    q = torch.randn(B, Hkv * G, 128, generator=g, device="cuda").to(torch.bfloat16)
    geom = rk.Geom(B, Hkv * G, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, cap, 16)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    got = {"deferred": [], "plain": []}
    try:
        for spin in (256, 0, 1, 2, 0, 256):
            rk.rk_debug_set_slice_spin(spin)
            for kind, runs in got.items():
                out, lse = torch.full_like(q, 7.0), torch.full((B, Hkv * G), 7.0, device="cuda")
                (rk.rk_full_attn_deferred if kind == "deferred" else rk.rk_full_attn)(geom, q, K, V, sl, cap, out, lse=lse, workspace=ws)
                torch.cuda.synchronize()
                runs.append((out.clone(), lse.clone()))
    finally:
        rk.rk_debug_set_slice_spin(256)
    for kind, runs in got.items():
        for out, lse in runs[1:]:
            assert torch.equal(out, runs[0][0]) and torch.equal(lse, runs[0][1]), kind
    for b, n in enumerate(lens[:3]):
        s = SCALE * torch.matmul(q[b].double().view(Hkv, G, 128), K[b, :, :n].double().transpose(1, 2).contiguous())
        ref = torch.matmul(torch.softmax(s, dim=-1), V[b, :, :n].double()).reshape(-1, 128)
        for kind, runs in got.items():
            d = (runs[0][0][b].double() - ref).abs()                   # one bf16 step of the larger value, and 4e-6 (see helpers)
            assert (d <= torch.maximum(runs[0][0][b].double().abs(), ref.abs()) * 2.0 ** -7 + 4e-6).all(), (kind, b)


# budgets around whole workgroups of 128 rows (the new token's row alone in a tile, in a workgroup of its own, or neither),
# beyond the 4096 rows the finishing kernel requests up front, few and many (sequence, KV head) pairs, empty, growing, full
# and over-full caches
H2O_EDGES = [("b127", 1, 4, 127, [127, 126, 0]), ("b128", 4, 2, 128, [128, 5]), ("b2047", 1, 8, 2047, [2047]), ("b2048_g7", 7, 4, 2048, [2048, 2000]),
             ("b4100", 4, 2, 4100, [4100]), ("b64_many", 2, 8, 64, [64, 63, 1, 0] * 4), ("b300_overfull", 3, 2, 300, [303, 300]),
             ("b5_g8", 8, 1, 5, [5, 2]), ("b700_g5", 5, 3, 700, [700]), ("b700_g6", 6, 3, 700, [699])]


@pytest.mark.parametrize("agg", [0, 1, 2], ids=["max", "mean", "first"])
@pytest.mark.parametrize("case", H2O_EDGES, ids=[c[0] for c in H2O_EDGES])
def test_h2o_step_equals_its_parts(rk, case, agg):
    """rk_h2o_step in its two launches against the same step on rows that are only 4-byte aligned, which goes through
    append, full attention and update one after the other: the same positions, rows and drops, totals to 2e-6 relative
    (the same fp32 weights from an lse whose fp64 sum is taken in another order), outputs to one bf16 step."""
    name, G, Hkv, budget, n0 = case
    say("h2o edge", name, agg)
    B, cap = len(n0), budget + 6
    g = torch.Generator(device="cuda").manual_seed(budget + agg)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    geom = rk.Geom(B, G * Hkv, Hkv, 128, SCALE)
    K, V = rnd(B, Hkv, cap, 128), rnd(B, Hkv, cap, 128)
    total = torch.rand(B, Hkv, cap, generator=g, device="cuda")
    pos = torch.stack([torch.stack([torch.randperm(cap, generator=g, device="cuda") for _ in range(Hkv)]) for _ in range(B)]).to(torch.int32)
    sides = []
    for _ in range(2):
        s = {"K": K.clone(), "V": V.clone(), "total": total.clone(), "pos": pos.clone(),
             "n_rows": torch.tensor(n0, dtype=torch.int32, device="cuda"), "n_attend": torch.zeros(B, dtype=torch.int32, device="cuda"),
             "out": torch.zeros(B, G * Hkv, 128, dtype=torch.bfloat16, device="cuda"),
             "dropped": torch.full((B, Hkv), -9, dtype=torch.int32, device="cuda"), "ws": rk.Workspace(geom, budget + 1, 1)}
        s["st"] = rk.h2o_state(geom, s["K"], s["V"], s["total"], s["pos"], s["n_rows"], s["n_attend"])
        sides.append(s)
    odd = torch.zeros(2, B * Hkv * 128 + 8, dtype=torch.bfloat16, device="cuda")
    for step in range(3):
        q, kn, vn = rnd(B, G * Hkv, 128), rnd(B, Hkv, 128), rnd(B, Hkv, 128)
        odd[0, 2:2 + kn.numel()], odd[1, 2:2 + kn.numel()] = kn.flatten(), vn.flatten()
        lens = torch.full((B,), cap + 1 + step, dtype=torch.int32, device="cuda")
        rk.rk_h2o_step(geom, sides[0]["st"], q, kn, vn, lens, budget, budget // 2, sides[0]["out"], agg=agg, dropped=sides[0]["dropped"], workspace=sides[0]["ws"])
        ko, vo = odd[0, 2:2 + kn.numel()].view(B, Hkv, 128), odd[1, 2:2 + kn.numel()].view(B, Hkv, 128)
        assert ko.data_ptr() % 16 != 0
        rk.rk_h2o_step(geom, sides[1]["st"], q, ko, vo, lens, budget, budget // 2, sides[1]["out"], agg=agg, dropped=sides[1]["dropped"], workspace=sides[1]["ws"])
        torch.cuda.synchronize()
        a, b = sides
        for key in ("K", "V", "pos", "n_rows", "n_attend", "dropped"):
            assert torch.equal(a[key], b[key]), (name, step, key)
        assert ((a["total"] - b["total"]).abs() <= 2e-6 * b["total"].abs()).all(), (name, step)
        x, y = a["out"].double(), b["out"].double()
        assert ((x - y).abs() <= torch.maximum(x.abs(), y.abs()) * 2.0 ** -7 + 4e-6).all(), (name, step)


# every sum of the merge of its own (up to 4 heads) and two to a thread (beyond), few and more than 64 partial results, shares by
# length, evenly over more sequences than are shared out, the new row alone in a tile and in the middle of one
H2O_BITS = [("batch4", 4, 8, 2048, [2048] * 4), ("ragged", 4, 8, 2048, [2048, 700, 1, 1999]), ("one", 4, 8, 2048, [2048]), ("g1_one_head_71_parts", 1, 1, 9000, [9000]),
            ("g5_ragged", 5, 2, 1500, [1500, 31, 640]), ("g7_130_parts", 7, 1, 16700, [16700]), ("g8", 8, 2, 700, [700, 699]), ("g2_70_sequences", 2, 2, 130, [130, 64] * 35),
            ("g3_overfull", 3, 2, 300, [303, 300]), ("g6", 6, 1, 31, [31])]


@pytest.mark.parametrize("aligned", [True, False])
@pytest.mark.parametrize("case", H2O_BITS, ids=[c[0] for c in H2O_BITS])
def test_h2o_step_has_the_bits_of_append_attention_update(rk, case, aligned):
    """rk_h2o_step against rk_h2o_append, rk_full_attn with its weights and rk_h2o_update called one after the other, over
    three steps: the same bits everywhere, output and totals among them."""
    name, G, Hkv, budget, n0 = case
    say("h2o bits", name, aligned)
    B, cap = len(n0), budget + 6
    g = torch.Generator(device="cuda").manual_seed(budget + G)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    geom = rk.Geom(B, G * Hkv, Hkv, 128, SCALE)
    K, V = rnd(B, Hkv, cap, 128), rnd(B, Hkv, cap, 128)
    total = torch.rand(B, Hkv, cap, generator=g, device="cuda")
    pos = torch.randperm(cap, generator=g, device="cuda").to(torch.int32).expand(B, Hkv, cap).contiguous()
    sides = []
    for _ in range(2):
        s = {"K": K.clone(), "V": V.clone(), "total": total.clone(), "pos": pos.clone(),
             "n_rows": torch.tensor(n0, dtype=torch.int32, device="cuda"), "n_attend": torch.zeros(B, dtype=torch.int32, device="cuda"),
             "out": torch.zeros(B, G * Hkv, 128, dtype=torch.bfloat16, device="cuda"),
             "dropped": torch.full((B, Hkv), -9, dtype=torch.int32, device="cuda"), "ws": rk.Workspace(geom, budget + 1, 1)}
        s["st"] = rk.h2o_state(geom, s["K"], s["V"], s["total"], s["pos"], s["n_rows"], s["n_attend"])
        sides.append(s)
    a, b = sides
    weights = torch.zeros(B, G * Hkv, budget + 1, device="cuda")
    room = torch.zeros(2, B * Hkv * 128 + 8, dtype=torch.bfloat16, device="cuda")
    for step in range(3):
        q, new = rnd(B, G * Hkv, 128), rnd(2, B, Hkv, 128)
        at = 0 if aligned else 2
        room[:, at:at + new[0].numel()] = new.view(2, -1)
        kn, vn = (room[i, at:at + new[0].numel()].view(B, Hkv, 128) for i in range(2))
        assert (kn.data_ptr() % 16 == 0 and vn.data_ptr() % 16 == 0) == aligned
        lens = torch.full((B,), cap + 1 + step, dtype=torch.int32, device="cuda")
        rk.rk_h2o_step(geom, a["st"], q, kn, vn, lens, budget, budget // 2, a["out"], dropped=a["dropped"], workspace=a["ws"])
        rk.rk_h2o_append(geom, b["st"], kn, vn, lens, budget)
        rk.rk_full_attn(geom, q, b["K"], b["V"], b["n_attend"], budget + 1, b["out"], weights=weights, workspace=b["ws"])
        rk.rk_h2o_update(geom, b["st"], weights, budget, budget // 2, dropped=b["dropped"])
        torch.cuda.synchronize()
        for key in ("K", "V", "pos", "n_rows", "n_attend", "dropped", "total", "out"):
            assert torch.equal(a[key], b[key]), (name, step, key)


@pytest.mark.parametrize("B", [24, 25], ids=["up_to_192MB", "beyond_192MB"])
def test_batched_gather_of_large_small_caches(rk, B):
    """The batched gather on both sides of the size from which it stores past the caches: bit copies of the selected
    rows, slots without a row left alone."""
    say("large batched gather", B)
    import ctypes
    Hkv, k, n = 8, 2048, 2060
    g = torch.Generator(device="cuda").manual_seed(B)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16)
    K, V, q = rnd(B, Hkv, n, 128), rnd(B, Hkv, n, 128), rnd(B, Hkv, 128)
    lens = torch.full((B,), n, dtype=torch.int32, device="cuda")
    lens[1] = k - 7                                      # fewer rows than slots
    geom = rk.Geom(B, Hkv, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, n, k)
    sK, sV = torch.full((B, Hkv, k, 128), 3.0, dtype=torch.bfloat16, device="cuda"), torch.full((B, Hkv, k, 128), 5.0, dtype=torch.bfloat16, device="cuda")
    idx, tail = torch.zeros(B, Hkv, k, dtype=torch.int32, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
    state = rk.layer_state(geom, K, V, sK, sV, idx, tail, k=k)
    rk.rk_full_attn_deferred(geom, q, K, V, lens, n, torch.empty_like(q), workspace=ws)
    rk.rk_refresh_batched(geom, (type(state) * 1)(state), (ctypes.c_void_p * 1)(ws.ptr), ws.nbytes, lens, n, k, pool_w=7)
    torch.cuda.synchronize()
    at = idx.long().clamp(min=0)[..., None].expand(-1, -1, -1, 128)
    there = (idx >= 0)[..., None]
    assert int((idx < 0).sum()) == 7 * Hkv and torch.equal(tail, lens)
    assert torch.equal(sK, torch.where(there, torch.gather(K, 2, at), torch.full_like(sK, 3.0)))
    assert torch.equal(sV, torch.where(there, torch.gather(V, 2, at), torch.full_like(sV, 5.0)))


# One tile per workgroup: 64 rows (16 per wavefront) up to 256 workgroups, 128 rows beyond, in up to 65 partial results (merged in
# units of 16, 8 and 4 rows, by up to 20, 40 and more of them), a workgroup or more for the rows decoded since the refresh; and
# attn_split_kernel where that ends.  Per sequence: (tail_start, rows since).
TILE_EDGES = [("k1", 4, 8, 1, 4, 0, [(900, 3)]), ("k16_17_g1", 1, 3, 17, 4, 0, [(900, 4), (16, 1)]), ("k63_g8", 8, 2, 63, 70, 0, [(900, 65), (900, 64), (62, 0)]),
              ("k64_g5", 5, 2, 64, 8, 0, [(64, 8), (63, 7), (0, 2), (0, 0)]), ("k65_evict", 4, 4, 65, 40, 1, [(900, 40), (900, 1), (900, 0)]),
              ("k256_evicts_all", 2, 2, 256, 300, 1, [(900, 300), (900, 256), (900, 129)]), ("none_selected", 4, 2, 0, 200, 0, [(900, 200), (500, 0), (0, 129)]),
              ("k1280_20_chunks", 3, 2, 1280, 5, 0, [(1279, 5), (2000, 0)]), ("k2560_g7", 7, 2, 2560, 5, 0, [(2560, 5)]), ("k2561_u4", 4, 4, 2561, 1, 0, [(3000, 1)]),
              ("k4096_65_chunks_g7", 7, 4, 4096, 64, 0, [(4096, 64)]), ("k4096_8w", 4, 8, 4096, 5, 0, [(4096, 5)]), ("two_17_g6", 6, 8, 4100, 128, 0, [(4100, 128)]),
              ("two_32_g8", 8, 4, 8192, 100, 0, [(8192, 100)]), ("k7900_63_chunks_8w_g7", 7, 4, 7900, 9, 0, [(7900, 9)]), ("k3900_8w_g8", 8, 8, 3900, 5, 0, [(3900, 5)]), ("k8192_split", 4, 8, 8192, 5, 0, [(8192, 5)]),
              ("batch", 4, 8, 700, 9, 0, [(700 + 37 * b, b) for b in range(9)]), ("batch_3_per_cu", 4, 8, 512, 9, 0, [(600, 9 - b % 4) for b in range(16)]),
              # groups beyond 4 over more than 16 pairs: partial results with maximum and sum apart
              ("exact_g7", 7, 4, 300, 9, 0, [(700 + 37 * b, b) for b in range(6)]), ("exact_g8_8w", 8, 8, 500, 9, 0, [(505, 9 - b) for b in range(7)]),
              ("two_exact_g5_11", 5, 1, 2800, 5, 1, [(2790 + b, 5) for b in range(17)]), ("exact_g5_25_chunks", 5, 4, 3070, 5, 0, [(3065 + b, 5 - b) for b in range(5)]), ("exact_g6_empty", 6, 9, 70, 70, 0, [(0, 0), (0, 70), (200, 0)])]
# Two tiles to a wavefront (test_launch_sizes has the form that each of the list takes): rows since in workgroups of their own and in the slots behind the small
# cache's, where that ends inside a tile, at its edge, at a wavefront's and a workgroup's; cached rows fewer than K; up to 64 results.
TILE_EDGES += [("two_own_tail", 4, 8, 6000, 11, 0, [(6000, 11)]), ("two_inside_8150", 4, 8, 8150, 40, 0, [(8190, 40)]), ("two_inside_fixed", 4, 8, 8192, 300, 1, [(8200, 300)]),
               ("two_inside_fixed_17", 4, 8, 8192, 20, 1, [(8200, 17)]), ("two_inside_fixed_256", 4, 8, 8192, 256, 1, [(8200, 256)]), ("two_batch", 4, 8, 2000, 48, 0, [(2100, 48), (1999, 16), (1008, 33), (0, 7)]), ("two_batch_fixed", 3, 8, 2048, 32, 1, [(2100, 32), (2048, 31), (1000, 0), (5, 16)]),
               ("two_512", 4, 8, 1700, 9, 0, [(1690 + 10 * b, 9 - b) for b in range(8)]), ("two_g7_64_results", 7, 4, 16000, 250, 0, [(16010, 250)]), ("two_exact_g8", 8, 8, 1900, 60, 0, [(1900, 60), (1800, 59), (40, 1), (3000, 0)]),
               ("two_exact_g5_fixed", 5, 8, 1536, 9, 1, [(1600, 9 - b) for b in range(5)]), ("two_g1", 1, 8, 4000, 30, 0, [(4000, 30), (100, 30)])]
# ... their second tiles, the small cache's second half, requested once the lengths are known: rows that end in either half, at its edge and a tile's, rows
# since in one tile, over the edge and in workgroups of their own, fewer selected rows than evicted ones.
TILE_EDGES += [("late_halves", 4, 8, 1700, 9, 0, [(896, 0), (895, 9), (880, 9), (897, 0), (1700, 9), (0, 5), (0, 0), (17, 1)]), ("late_2_of_440", 4, 8, 440, 16, 0, [(440 - 23 * b, b) for b in range(16)]),
               ("late_fixed_300", 4, 8, 1000, 300, 1, [(1000, 300), (900, 299), (700, 150), (512, 0), (1000, 1), (300, 300), (0, 300), (1100, 44)]),
               ("late_exact_g5_24_results", 5, 4, 6100, 9, 0, [(6100, 9), (3000, 2), (6109, 0), (6090, 8), (100, 1)]), ("late_exact_g7_own_tail", 7, 4, 5880, 9, 0, [(5880 + b, 9 - b) for b in range(5)]),
               ("late_g8_15", 8, 8, 3600, 20, 0, [(3600, 20), (1920, 20), (3700, 0), (1905, 17)])]


@pytest.mark.parametrize("case", TILE_EDGES, ids=[c[0] for c in TILE_EDGES])
def test_partial_step_at_tile_edges(rk, case):
    """Against fp64, one bf16 step of the larger value and 4e-6 (see helpers); the bits do not depend on who merges (bound on the
    re-reads of rows in flight at 0, 1, default), nor does NaN past the rows of a sequence; strided caches, out 2-byte aligned."""
    name, G, Hkv, k, max_recent, evict, seqs = case
    say("tile edge", name)
    B, cap = len(seqs), max(t + r for t, r in seqs) + 2
    g = torch.Generator(device="cuda").manual_seed(k + G)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    K, V = rnd(B, Hkv, cap, 128), rnd(B, Hkv, cap, 128)
    sK, sV = rnd(B, Hkv, max(k, 1) + 3, 128), rnd(B, Hkv, max(k, 1) + 3, 128)
    q = rnd(B, Hkv * G, 128)
    rows, nan = [], float("nan")
    for b, (t0, r) in enumerate(seqs):
        n1 = min(max(k - (r if evict else 0), 0), t0)
        rows.append((n1, t0, t0 + r))
        sK[b, :, n1:], sV[b, :, n1:] = nan, nan
        K[b, :, :t0], V[b, :, :t0], K[b, :, t0 + r:], V[b, :, t0 + r:] = nan, nan, nan, nan
    geom = rk.Geom(B, Hkv * G, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, cap, max(k, 16))
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device="cuda")
    tail, lens = i32([t for t, _ in seqs]), i32([t + r for t, r in seqs])
    outs = []
    try:
        for spin in (256, 0, 1, 256):
            rk.rk_debug_set_slice_spin(spin)
            buf = torch.full((B * Hkv * G * 128 + 1,), 7.0, dtype=torch.bfloat16, device="cuda")
            out = buf[1:].view(B, Hkv * G, 128)
            fn = rk.rk_partial_attn_fixed if evict else rk.rk_partial_attn
            fn(geom, q, sK, sV, k, K, V, tail, lens, max_recent, out, workspace=ws)
            torch.cuda.synchronize()
            outs.append(out.clone())
    finally:
        rk.rk_debug_set_slice_spin(256)
    for o in outs[1:]:
        assert torch.equal(o, outs[0])
    for b, (n1, t0, n) in enumerate(rows):
        if n1 + n - t0 == 0:
            assert (outs[0][b] == 0).all()
            continue
        Kb = torch.cat([sK[b, :, :n1], K[b, :, t0:n]], dim=1).double()
        Vb = torch.cat([sV[b, :, :n1], V[b, :, t0:n]], dim=1).double()
        s = SCALE * torch.matmul(q[b].double().view(Hkv, G, 128), Kb.transpose(1, 2).contiguous())
        ref = torch.matmul(torch.softmax(s, dim=-1), Vb).reshape(-1, 128)
        d = (outs[0][b].double() - ref).abs()
        assert (d <= torch.maximum(outs[0][b].double().abs(), ref.abs()) * 2.0 ** -7 + 4e-6).all(), (b, float(d.max()))


# (heads per group, KV heads, sequences, rows of a workgroup)
TILE_WEIGHTS = [(7, 4, 6, 64), (8, 8, 4, 64), (5, 4, 16, 128), (6, 8, 9, 128)]


@pytest.mark.parametrize("shape", TILE_WEIGHTS, ids=["g%d_%dx%d_%d" % c for c in TILE_WEIGHTS])
def test_partial_step_weighs_its_workgroups_exactly(rk, shape):
    """Groups beyond 4 over more than 16 pairs: three workgroups whose sums are 1, 3/4 and 1/4 of a workgroup's rows with the same score
    of several hundred, values +1, -1 and -1.  The output is exactly 0; weights that went through a rounded log-sum-exp leave about
    1e-5 (scores of 400) and more."""
    G, Hkv, B, wg = shape
    say("tile weights", *shape)
    k = 3 * wg
    q = torch.ones(B, Hkv * G, 128, dtype=torch.bfloat16, device="cuda") * (1 + torch.arange(Hkv * G, device="cuda") / 16).to(torch.bfloat16)[:, None]
    sK = torch.zeros(B, Hkv, k, 128, dtype=torch.bfloat16, device="cuda")
    sV = torch.full_like(sK, 5.0)                             # rows of score 0 weigh e^-400: nothing
    for rows, value in ((slice(0, wg), 1.0), (slice(wg, wg + 3 * wg // 4), -1.0), (slice(2 * wg, 2 * wg + wg // 4), -1.0)):
        sK[:, :, rows], sV[:, :, rows] = 35.0 + torch.arange(Hkv, device="cuda")[:, None, None] / 4, value
    K = torch.full((B, Hkv, k + 4, 128), float("nan"), dtype=torch.bfloat16, device="cuda")
    geom = rk.Geom(B, Hkv * G, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, k + 4, k)
    lens = torch.full((B,), k, dtype=torch.int32, device="cuda")
    out = torch.full((B, Hkv * G, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    rk.rk_partial_attn(geom, q, sK, sV, k, K, K, lens, lens, 4, out, workspace=ws)
    torch.cuda.synchronize()
    say("largest output %.3g" % out.float().abs().max().item())
    assert (out == 0).all()


# The triggered step in each of its kernels: one tile per workgroup of 4 and 8 wavefronts, with a log-sum-exp and with (max, sum) pairs,
# and, where nine wavefronts to a workgroup would not all be resident, attn_split_kernel in its tagged and its ticketed form
# (test_launch_sizes asserts which takes which).  (heads per group, KV heads, sequences, K, bound on the rows since, fixed size)
TRIGGERED = {"tile_4w": (4, 8, 1, 2048, 5, False), "tile_4w_g8": (8, 4, 3, 700, 16, True), "tile_8w": (4, 8, 4, 1024, 9, True), "tile_8w_g7": (7, 4, 4, 1100, 5, False),
             "tile_8w_exact_g8": (8, 8, 4, 700, 9, False), "split_tagged_long": (4, 8, 1, 8192, 5, False), "split_tagged_batch": (4, 8, 4, 2048, 5, True),
             "split_tagged_g8": (8, 8, 1, 4096, 5, False), "split_ticketed_g7": (7, 4, 8, 1024, 5, True)}


@pytest.mark.parametrize("name", list(TRIGGERED))
def test_triggered_step_in_each_form(rk, name):
    """Outputs of the sequences that do not fire against fp64 (one bf16 step of the larger value and 4e-6), the others' untouched; sim, decision
    and reference as rk_query_sim has them; the same bits whoever merges and however often it is called."""
    G, Hkv, B, k, recent, fixed = TRIGGERED[name]
    say("triggered", name)
    Hq, cap = G * Hkv, k + 40
    g = torch.Generator(device="cuda").manual_seed(k + G + B)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    K, V, sK, sV, q = rnd(B, Hkv, cap, 128), rnd(B, Hkv, cap, 128), rnd(B, Hkv, k, 128), rnd(B, Hkv, k, 128), rnd(B, Hq, 128)
    ref = q.float().mean(1) * 2
    ref[1::2] = torch.randn(ref[1::2].shape, generator=g, device="cuda")
    since = [min(recent, 5 - b % 4) for b in range(B)]
    lens = torch.tensor([cap - 2 - b for b in range(B)], dtype=torch.int32, device="cuda")
    tail = lens - torch.tensor(since, dtype=torch.int32, device="cuda")
    geom = rk.Geom(B, Hq, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, cap, k)
    i32 = lambda: torch.full((B,), -1, dtype=torch.int32, device="cuda")
    ref_a, sim_a, need_a = ref.clone(), torch.zeros(B, device="cuda"), i32()
    rk.rk_query_sim(geom, q, ref_a, 0.5, False, sim_a, need_a)
    torch.cuda.synchronize()
    fired = need_a.bool().tolist()
    assert fired == [b % 2 == 1 for b in range(B)]
    outs = []
    try:
        for spin in (256, 0, 1, 256):
            rk.rk_debug_set_slice_spin(spin)
            out = torch.full((B, Hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
            ref_b, sim_b, need_b = ref.clone(), torch.zeros(B, device="cuda"), i32()
            rk.rk_partial_attn_triggered(geom, q, sK, sV, k, K, V, tail, lens, recent, out, ref_b, 0.5, sim_b, need_b, fixed_size=fixed, workspace=ws)
            torch.cuda.synchronize()
            assert torch.equal(sim_b, sim_a) and torch.equal(need_b, need_a) and torch.equal(ref_b, ref_a)
            outs.append(out)
    finally:
        rk.rk_debug_set_slice_spin(256)
    for o in outs[1:]:
        assert torch.equal(o, outs[0])
    for b in range(B):
        if fired[b]:
            assert (outs[0][b] == 7.0).all()
            continue
        n1, n, t0 = k - (since[b] if fixed else 0), int(lens[b]), int(tail[b])
        Kb = torch.cat([sK[b, :, :n1], K[b, :, t0:n]], dim=1).double()
        Vb = torch.cat([sV[b, :, :n1], V[b, :, t0:n]], dim=1).double()
        x = SCALE * torch.matmul(q[b].double().view(Hkv, G, 128), Kb.transpose(1, 2).contiguous())
        want = torch.matmul(torch.softmax(x, dim=-1), Vb).reshape(-1, 128)
        d = (outs[0][b].double() - want).abs()
        assert (d <= torch.maximum(outs[0][b].double().abs(), want.abs()) * 2.0 ** -7 + 4e-6).all(), (b, float(d.max()))


# Test steps in one launch (both branches; test_launch_sizes asserts which take it).  (heads per group, KV heads, rows, K, rows since, fixed
# size).  Full passes of 512 and of 256 workgroups, few partial results, rows fewer than K, more workgroups for the partial step than for the full pass.
TEST_STEPS = [(4, 8, 33000, 2048, 5, False), (4, 8, 45001, 2048, 5, True), (7, 4, 66000, 4096, 3, False), (7, 4, 9001, 700, 60, True),
              (8, 4, 2049, 128, 1, False), (1, 8, 3000, 256, 7, True), (2, 8, 700, 64, 16, False), (3, 4, 130, 64, 2, False),
              (5, 8, 4000, 500, 9, False), (6, 3, 1000, 1000, 4, False), (4, 4, 50, 64, 3, False), (7, 8, 8192, 2047, 130, False),
              (4, 8, 33000, 4096, 5, False), (7, 4, 20000, 4096, 140, True), (4, 8, 20000, 3001, 9, True), (8, 8, 9000, 4033, 1, False), (2, 8, 5000, 8000, 3, False)]
TEST_STEPS_128 = 5                             # the last ones: 128 rows to a workgroup, where the call of its own shares them out another way


@pytest.mark.parametrize("case", TEST_STEPS, ids=["g%d_%dx%d_k%d_r%d" % c[:5] for c in TEST_STEPS])
def test_test_step_in_one_launch(rk, case):
    """The bits (or, with 128 rows to a workgroup, the partial step's to a step of bf16) of the partial step with its test and then the full pass
    under the decision, as calls of their own: layers that fire and layers that do not, whoever merges, call after call."""
    G, Hkv, n, k, recent, fixed = case
    say("test step", case)
    layers, Hq, cap = 3, G * Hkv, n + 8
    g = torch.Generator(device="cuda").manual_seed(n + k)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda")
    kv = [(rnd(1, Hkv, cap, 128).to(torch.bfloat16), rnd(1, Hkv, cap, 128).to(torch.bfloat16)) for _ in range(layers)]
    geom = rk.Geom(1, Hq, Hkv, 128, SCALE)
    q0 = rnd(layers, 1, Hq, 128).to(torch.bfloat16)
    models = []
    for _ in range(2):
        lens = torch.tensor([n - recent], dtype=torch.int32, device="cuda")
        m = rk.RefreshKVModel(geom, kv, lens, n - recent, k, 4, dynamic=True, threshold=0.9, evict_lowest=fixed)
        m.batched_refresh()
        m.step(0, q0)
        lens += recent
        for _ in range(recent):
            m.advance()
        models.append(m)
    one, two = models
    try:
        for t, spin, fires in ((4, 256, [0, 1, 0]), (8, 0, [1, 0, 1]), (12, 1, [0, 0, 0]), (16, 2, [1, 1, 1]), (20, 256, [0, 1, 1])):
            rk.rk_debug_set_slice_spin(spin)
            q = torch.stack([rnd(1, Hq, 128).to(torch.bfloat16) if f else
                             (m_ref[None, None] + 0.01 * rnd(1, Hq, 128)).to(torch.bfloat16) for f, m_ref in zip(fires, one.q_ref[:, 0])])
            for m in models:
                m.out.fill_(7.0)
            assert one.step(t, q) == "both"
            for l in range(layers):
                K, V = kv[l]
                rk.rk_partial_attn_triggered(geom, q[l], two.small_K[l], two.small_V[l], k, K, V, two.tail_start[l], two.seq_lens, max(recent, 1),
                                             two.out[l], two.q_ref[l], 0.9, two.sim[l], two.need_full[l], fixed_size=fixed, workspace=two._wss[l])
                rk.rk_full_attn_deferred(geom, q[l], K, V, two.seq_lens, n, two.out[l], pred=two.need_full[l], pred_val=1, workspace=two._wss[l])
            rk.rk_refresh_batched(geom, two._layers, two._batched_ptrs, two._batched_bytes, two.seq_lens, n, k, pool_w=7, by_need_full=True)
            torch.cuda.synchronize()
            assert one.need_full[:, 0].tolist() == fires
            for name in ("need_full", "sim", "q_ref", "tail_start", "n_full"):
                assert torch.equal(getattr(one, name), getattr(two, name)), name
            assert torch.equal(one.idx, two.idx) and torch.equal(one.small_K, two.small_K) and torch.equal(one.small_V, two.small_V)
            a, b = one.out.double(), two.out.double()
            for l in range(layers):
                if fires[l] or case not in TEST_STEPS[-TEST_STEPS_128:]:
                    assert torch.equal(a[l], b[l]), l
                else:      # sums in another order: a step of bf16 of the larger value, and 4e-6
                    assert ((a[l] - b[l]).abs() <= torch.maximum(a[l].abs(), b[l].abs()) * 2.0 ** -7 + 4e-6).all(), l
    finally:
        rk.rk_debug_set_slice_spin(256)


# (heads per group, KV heads, sequences, rows, K): tiles of 4 and 8 wavefronts, their last one partly filled, pairs and log-sum-exps as weights, more
# ranks than rows, and more rows than are resident at once (two launches).
GATHER_ATTN = [(4, 8, 1, 9000, 8192), (4, 8, 1, 3000, 2048), (4, 8, 1, 3000, 65), (7, 4, 1, 5000, 4097), (1, 8, 1, 500, 1), (3, 3, 2, 700, 127), (8, 4, 1, 90, 200),
               (4, 8, 4, 2100, 1025), (7, 4, 6, 1300, 512), (5, 8, 3, 1000, 300), (2, 8, 5, 3000, 2500), (6, 8, 16, 700, 350), (8, 8, 4, 1200, 900)]


@pytest.mark.parametrize("case", GATHER_ATTN, ids=["g%d_%dx%d_n%d_k%d" % (c[0], c[2], c[1], c[3], c[4]) for c in GATHER_ATTN])
def test_gather_inside_the_step(rk, case):
    """Small caches (strided, of more than K rows) and tail_start bit for bit as the gather leaves them, rows without an entry untouched; outputs against fp64 (one bf16 step
    of the larger value and 4e-6); a sequence that the predicate leaves out stays as it is."""
    G, Hkv, B, n, k = case
    say("gather inside", case)
    Hq, cap = G * Hkv, n + 6
    g = torch.Generator(device="cuda").manual_seed(n + k)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    K, V, q = rnd(B, Hkv + 1, cap + 3, 128)[:, 1:, :cap], rnd(B, Hkv + 1, cap + 3, 128)[:, 1:, :cap], rnd(B, Hq, 128)      # heads and rows that are others'
    lens = torch.tensor([n - 37 * (b % 2) for b in range(B)], dtype=torch.int32, device="cuda")
    idx = torch.full((B, Hkv, k), -1, dtype=torch.int32, device="cuda")
    for b in range(B):
        m = min(k, int(lens[b]))
        idx[b, :, :m] = torch.stack([torch.randperm(int(lens[b]), generator=g, device="cuda")[:m] for _ in range(Hkv)]).to(torch.int32)
    geom = rk.Geom(B, Hq, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, cap, k)
    pred = torch.tensor([0 if b == 1 else 1 for b in range(B)], dtype=torch.int32, device="cuda")
    for use_pred, spin in ((False, 256), (True, 0), (True, 256)):
        p = pred if use_pred else None
        rk.rk_debug_set_slice_spin(spin)
        try:
            small = [[torch.full((B, Hkv + 2, k + 5, 128), 3.0, dtype=torch.bfloat16, device="cuda") for _ in range(2)] for _ in range(2)]
            state = [[t[:, 1:-1] for t in pair] + [torch.full((B,), 5, dtype=torch.int32, device="cuda")] for pair in small]
            rk.rk_gather_small_kv(geom, K, V, idx, k, state[0][0], state[0][1], seq_lens=lens, tail_start=state[0][2], pred=p, pred_val=1)
            out = torch.full((B, Hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
            rk.rk_gather_attn(geom, q, K, V, idx, k, state[1][0], state[1][1], lens, state[1][2], out, pred=p, pred_val=1, workspace=ws)
            torch.cuda.synchronize()
        finally:
            rk.rk_debug_set_slice_spin(256)
        for a, b in zip(small[0] + state[0][2:], small[1] + state[1][2:]):
            assert torch.equal(a, b)
        for b in range(B):
            if use_pred and b == 1:
                assert (out[b] == 7.0).all()
                continue
            m = min(k, int(lens[b]))
            at = idx[b, :, :m].long()[:, :, None].expand(-1, -1, 128)
            Kb, Vb = torch.gather(K[b], 1, at).double(), torch.gather(V[b], 1, at).double()
            x = SCALE * torch.matmul(q[b].double().view(Hkv, G, 128), Kb.transpose(1, 2).contiguous())
            want = torch.matmul(torch.softmax(x, dim=-1), Vb).reshape(-1, 128)
            d = (out[b].double() - want).abs()
            assert (d <= torch.maximum(out[b].double().abs(), want.abs()) * 2.0 ** -7 + 4e-6).all(), (b, float(d.max()))


# What the C++ checks leave to binding.py: the calls, in order gather, partial, fixed, partial with a predicate, full, full with lse and a predicate, H2O
MARSHALLED = {"plain": "", "strided": "", "parameter": "", "stream": "", "subclass": "partial fixed pred full lse h2o", "numpy_int": "gather partial fixed pred",
              "wrong_shape": "partial fixed pred full lse h2o", "wrong_type": "partial fixed pred full lse h2o", "not_contiguous": "partial fixed pred full lse h2o",
              "short_cache": "gather partial fixed pred", "not_a_state": "h2o"}


class _Sub(torch.Tensor):
    pass


@pytest.mark.parametrize("form", list(MARSHALLED))
def test_calls_marshalled_in_cpp_take_what_python_takes(rk, form, monkeypatch):
    """The same results, or the same exception, whether the arguments go through the C++ checks or through those of binding.py alone; the common case goes
    through C++, and what is not does not."""
    B, G, Hkv, n, k = 2, 4, 3, 300, 64
    g = torch.Generator(device="cuda").manual_seed(5)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda").to(torch.bfloat16)
    geom = rk.Geom(B, G * Hkv, Hkv, 128, SCALE)
    K, V, q = rnd(B, Hkv, n, 128), rnd(B, Hkv, n, 128), rnd(B, G * Hkv, 128)
    new = rnd(2, B, Hkv, 128)
    idx = torch.stack([torch.randperm(n - 9, generator=g, device="cuda")[:k] for _ in range(B * Hkv)]).view(B, Hkv, k).to(torch.int32)
    n_sel, stream = k, None
    if form == "strided":
        K, V = rnd(B, Hkv + 2, n + 5, 128)[:, 1:-1, :n], rnd(B, Hkv + 2, n + 5, 128)[:, 1:-1, :n]
    elif form == "parameter":
        q = torch.nn.Parameter(q, requires_grad=False)
    elif form == "subclass":
        q = q.as_subclass(_Sub)
    elif form == "numpy_int":
        n_sel = np.int64(k)
    elif form == "stream":
        stream = torch.cuda.Stream()
    elif form == "wrong_shape":
        q = q[:, :-1].contiguous()
    elif form == "wrong_type":
        q = q.float()
    elif form == "not_contiguous":
        q = rnd(B, 128, G * Hkv).transpose(1, 2)
    elif form == "short_cache":
        n_sel = k + 1

    def run():
        ws = rk.Workspace(geom, n, k)
        lens, tail = torch.tensor([n, n - 7], dtype=torch.int32, device="cuda"), torch.tensor([n - 9, n - 9], dtype=torch.int32, device="cuda")
        sK, sV = torch.zeros(2, B, Hkv, k, 128, dtype=torch.bfloat16, device="cuda")
        total, pos = torch.ones(B, Hkv, n, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda").expand(B, Hkv, n).contiguous()
        cache = [t.clone().contiguous() for t in (K, V)]
        n_rows, n_attend = torch.full((B,), n - 1, dtype=torch.int32, device="cuda"), torch.zeros(B, dtype=torch.int32, device="cuda")
        state = rk.h2o_state(geom, *cache, total, pos, n_rows, n_attend)
        if form == "not_a_state":
            state = bytes(state)           # as long as the structure, but not one
        outs = [torch.zeros(B, G * Hkv, 128, dtype=torch.bfloat16, device="cuda") for _ in range(6)]
        pred, lse, dropped = torch.tensor([1, 0], dtype=torch.int32, device="cuda"), torch.zeros(B, G * Hkv, device="cuda"), torch.full((B, Hkv), -9, dtype=torch.int32, device="cuda")
        if stream is not None:
            stream.wait_stream(torch.cuda.current_stream())
        res = {}
        for name, call in (("gather", lambda: rk.rk_gather_small_kv(geom, K, V, idx, n_sel, sK, sV, seq_lens=lens, tail_start=tail.clone() if stream is None else None, stream=stream)),
                           ("partial", lambda: rk.rk_partial_attn(geom, q, sK, sV, n_sel, K, V, tail, lens, 16, outs[0], workspace=ws, stream=stream)),
                           ("fixed", lambda: rk.rk_partial_attn_fixed(geom, q, sK, sV, n_sel, K, V, tail, lens, 16, outs[1], workspace=ws, stream=stream)),
                           ("pred", lambda: rk.rk_partial_attn(geom, q, sK, sV, n_sel, K, V, tail, lens, 16, outs[2], pred=pred, pred_val=1, workspace=ws, stream=stream)),
                           ("full", lambda: rk.rk_full_attn(geom, q, K, V, lens, n, outs[3], workspace=ws, stream=stream)),
                           ("lse", lambda: rk.rk_full_attn(geom, q, K, V, lens, n, outs[4], lse=lse, pred=pred, pred_val=0, workspace=ws, stream=stream)),
                           ("h2o", lambda: rk.rk_h2o_step(geom, state, q, new[0], new[1], lens, n - 1, n // 2, outs[5], dropped=dropped, workspace=ws, stream=stream))):
            try:
                call()
                res[name] = None
            except (ValueError, ctypes.ArgumentError) as e:
                res[name] = str(e)
        torch.cuda.synchronize()
        return res, [sK, sV, *outs, lse, dropped, total, pos, *cache, n_rows]

    taken = []

    def watched(call):
        def f(*a):
            taken.append(call(*a) is not None)
            return 0 if taken[-1] else None                   # (every call that C++ takes here succeeds)
        return f
    names = ("rk_gather_small_kv", "rk_partial_attn", "rk_partial_attn_fixed", "rk_full_attn", "rk_h2o_step")
    native = rk.binding._native
    monkeypatch.setattr(rk.binding, "_native", type("watched", (), {name: staticmethod(watched(getattr(native, name))) for name in names}))
    by_cpp = run()
    monkeypatch.setattr(rk.binding, "_native", type("none", (), {name: staticmethod(lambda *a: None) for name in names}))
    by_python = run()
    assert by_cpp[0] == by_python[0], (by_cpp[0], by_python[0])
    assert [name for name, t in zip(by_cpp[0], taken) if not t] == MARSHALLED[form].split() and len(taken) == len(by_cpp[0])
    assert any(by_cpp[0].values()) == (form in ("wrong_shape", "wrong_type", "not_contiguous", "short_cache", "not_a_state"))
    for a, b in zip(by_cpp[1], by_python[1]):
        assert torch.equal(a, b)


def _select_scores(name, rows, n, g):
    w = torch.exp(torch.randn(*rows, n, generator=g) * 1.2 - 10)
    if name == "levels":                   # few values: stretches do not fit, the row is one workgroup's
        w = torch.round(w * 2.0 ** 17) * 2.0 ** -17
    elif name == "equal":
        w = torch.full_like(w, 0.25)
    elif name == "mostly_zero":
        w = torch.where(torch.rand(*rows, n, generator=g) < 0.01, w, torch.zeros_like(w))
    elif name == "one_bin":                # all scores in one bin of the histogram
        w = 1.0 + 0.1 * torch.rand(*rows, n, generator=g)
    elif name == "narrow":                 # a few bins with many times K positions each
        w = torch.exp(torch.randn(*rows, n, generator=g) * 0.05 - 10)
    elif name == "narrow2":
        w = torch.exp(torch.randn(*rows, n, generator=g) * 0.25 - 10)
    elif name == "steps":                  # ... in which scores come in clusters
        w = (1.0 + 0.25 * torch.rand(*rows, n, generator=g).mul(5).floor() / 5) * (1 + 2.0 ** -16 * torch.rand(*rows, n, generator=g))
    elif name == "infinite":
        w[..., 5], w[..., n // 2] = float("inf"), float("inf")
    return w


# (scores, B, Hkv, n, k, pool): 8 / 4 / 2 / 1 workgroups per row, fewer ranks than workgroups, fewer positions than ranks, vectors of
# four and rounds of 32768 positions that end in the row, more than 256 runs in a stretch; bins with more than four times K positions,
# which a part looks into ("narrow", "one_bin", "steps")
SELECT_EDGES = [("normal", 1, 1, 1, 1, 1), ("normal", 1, 2, 9, 3, 7), ("normal", 1, 3, 31, 100, 7), ("normal", 1, 8, 1027, 9, 1), ("normal", 2, 16, 4099, 300, 7),
                ("normal", 5, 8, 5001, 700, 3), ("normal", 16, 8, 3001, 257, 7), ("normal", 33, 8, 1025, 64, 7), ("normal", 1, 8, 32771, 2048, 7),
                ("normal", 1, 4, 65537, 8192, 1), ("normal", 1, 2, 98305, 16384, 7), ("levels", 1, 8, 20001, 3000, 1), ("levels", 3, 8, 20001, 900, 7),
                ("equal", 1, 8, 5003, 500, 7), ("equal", 1, 4, 40001, 12000, 1), ("mostly_zero", 1, 8, 30001, 2000, 1), ("one_bin", 1, 8, 30001, 2000, 1),
                ("one_bin", 2, 8, 9001, 1000, 7), ("infinite", 1, 8, 9001, 300, 7), ("narrow", 1, 8, 2001, 125, 1), ("narrow", 1, 8, 33001, 1500, 7), ("narrow", 1, 1, 70003, 9, 1),
                ("narrow2", 1, 4, 131073, 8192, 7), ("narrow2", 3, 16, 9001, 500, 1), ("narrow2", 20, 8, 5001, 64, 7), ("steps", 1, 8, 20001, 1000, 1),
                ("steps", 1, 4, 40001, 4001, 1), ("steps", 2, 16, 5003, 100, 7),
                # few ranks: bins taken whole up to 256 positions, looked into beyond 1024, neither between
                ("narrow", 1, 9, 37291, 19, 7), ("normal", 1, 2, 25489, 1, 7), ("narrow", 4, 4, 521, 8, 7), ("one_bin", 1, 8, 257, 5, 1), ("one_bin", 1, 8, 1025, 5, 1),
                ("one_bin", 1, 8, 1023, 5, 1),
                # a few long rows: listed by a workgroup per 4096 positions, ranked by the last to arrive
                ("normal", 1, 1, 98304, 3, 1), ("normal", 3, 2, 98309, 4096, 7), ("normal", 1, 4, 163841, 8192, 1), ("normal", 1, 1, 327683, 16384, 7),
                ("levels", 2, 2, 98305, 2000, 1), ("equal", 1, 1, 98306, 500, 7), ("narrow", 1, 6, 100003, 1500, 7), ("mostly_zero", 2, 1, 98307, 2000, 1),
                ("infinite", 1, 3, 98305, 300, 7), ("normal", 1, 1, 49152, 3072, 7), ("normal", 4, 1, 49157, 1000, 1), ("infinite", 2, 1, 49153, 1500, 1),
                # ... shared out by rank after all, all of them or some (candidates that do not fit, not even as runs; thousands of runs), by one workgroup
                ("narrow", 1, 2, 49153, 3000, 1), ("narrow", 2, 3, 65537, 4096, 7), ("narrow2", 1, 4, 65539, 4096, 7), ("narrow2", 1, 1, 196611, 12288, 7),
                ("one_bin", 1, 1, 50001, 2000, 1), ("steps", 1, 3, 70001, 1100, 1), ("levels", 1, 2, 262147, 10000, 1), ("equal", 3, 1, 49155, 3000, 1),
                ("mostly_zero", 1, 5, 50003, 1000, 1)]


@pytest.mark.parametrize("case", SELECT_EDGES, ids=["%s_%dx%d_%d_k%d_w%d" % c for c in SELECT_EDGES])
def test_selection_shared_out_by_rank(rk, case):
    """Positions and scores exactly those of a stable sort, three calls in a row (the workspace is left clean), with rows shorter
    than the longest whose workspace holds NaN behind them."""
    name, B, Hkv, n, k, pool_w = case
    say("selection by rank", *case)
    g = torch.Generator().manual_seed(n + k)
    w = _select_scores(name, (B, Hkv), n, g)
    lens = [n if b == 0 else max(1, n - 7 * b) for b in range(B)]
    geom = rk.Geom(B, Hkv, Hkv, 128, SCALE)
    ws = rk.Workspace(geom, n, k)
    idx = torch.empty(B, Hkv, k, dtype=torch.int32, device="cuda")
    sel = torch.empty(B, Hkv, k, device="cuda")
    wd, ld = w.cuda(), torch.tensor(lens, dtype=torch.int32, device="cuda")
    full = torch.full((B,), n, dtype=torch.int32, device="cuda")
    if B > 1:
        rk.rk_topk_select(geom, torch.full_like(wd, float("nan")), full, n, k, pool_w, idx, workspace=ws)
    for _ in range(3):
        idx.fill_(-7)
        rk.rk_topk_select(geom, wd, ld, n, k, pool_w, idx, sel_scores=sel, workspace=ws)
        torch.cuda.synchronize()
        for b, m in enumerate(lens):
            P = torch.nn.functional.max_pool1d(w[b, :, :m], pool_w, stride=1, padding=pool_w // 2)
            v, i = torch.sort(P, dim=-1, descending=True, stable=True)
            kk = min(k, m)
            assert torch.equal(idx[b, :, :kk].cpu().long(), i[:, :kk]), (name, b)
            assert torch.equal(sel[b, :, :kk].cpu(), v[:, :kk]), (name, b)
            assert (idx[b, :, kk:] == -1).all() and (sel[b, :, kk:] == 0).all()


# (layers, B, Hkv, n, k, lengths, which (layer, sequence) refresh)
LISTED_BATCHES = [(2, 1, 3, 98304, 1000, [98304], None), (3, 2, 1, 98309, 300, [98309, 50], [[1, 1], [0, 1], [1, 0]]), (2, 1, 2, 163841, 8192, [163841], None),
                  (1, 1, 6, 98305, 4096, [98304], None)]


@pytest.mark.parametrize("case", LISTED_BATCHES, ids=["l%d_%dx%d_%d_k%d" % c[:5] for c in LISTED_BATCHES])
def test_batched_selection_of_few_long_rows(rk, case):
    """rk_refresh_batched where the rows of all layers are few and long: the positions that rk_full_attn_select takes layer by layer
    and that a stable sort of its weights gives; others untouched; three calls on the same workspaces."""
    import ctypes
    L, B, Hkv, n, k, lens, on = case
    say("few long rows, batched", *case[:5])
    g = torch.Generator(device="cuda").manual_seed(n + k)
    rnd = lambda *s: torch.randn(*s, generator=g, device="cuda", dtype=torch.bfloat16)
    K, V, q = rnd(L, B, Hkv, n, 128), rnd(L, B, Hkv, n, 128), rnd(L, B, Hkv * 2, 128)
    geom = rk.Geom(B, Hkv * 2, Hkv, 128, SCALE)
    sl = torch.tensor(lens, dtype=torch.int32, device="cuda")
    need = torch.tensor(on or [[1] * B] * L, dtype=torch.int32, device="cuda")
    wss = [rk.Workspace(geom, n, k) for _ in range(L)]
    sK, sV = torch.zeros(L, B, Hkv, k, 128, dtype=torch.bfloat16, device="cuda"), torch.zeros(L, B, Hkv, k, 128, dtype=torch.bfloat16, device="cuda")
    idx, tail = torch.full((L, B, Hkv, k), -5, dtype=torch.int32, device="cuda"), torch.zeros(L, B, dtype=torch.int32, device="cuda")
    states = [rk.layer_state(geom, K[l], V[l], sK[l], sV[l], idx[l], tail[l], need_full=need[l], k=k) for l in range(L)]
    out, one = torch.empty_like(q[0]), torch.full((B, Hkv, k), -5, dtype=torch.int32, device="cuda")
    w = torch.zeros(B, Hkv * 2, (n + 3) // 4 * 4, device="cuda")
    for _ in range(3):
        idx.fill_(-5)
        for l in range(L):
            rk.rk_full_attn_deferred(geom, q[l], K[l], V[l], sl, n, out, pred=need[l], pred_val=1, workspace=wss[l])
        rk.rk_refresh_batched(geom, (type(states[0]) * L)(*states), (ctypes.c_void_p * L)(*[x.ptr for x in wss]), wss[0].nbytes, sl, n, k, pool_w=7,
                              by_need_full=True)
        torch.cuda.synchronize()
        for l in range(L):
            rk.rk_full_attn_select(geom, q[l], K[l], V[l], sl, n, out, k, 7, one, weights=w, workspace=rk.Workspace(geom, n, k))
            for b in range(B):
                if need[l, b].item() == 0:
                    assert (idx[l, b] == -5).all() and (sK[l, b] == 0).all()
                    continue
                assert torch.equal(idx[l, b], one[b]), (l, b)
                kk = min(k, lens[b])
                P = torch.nn.functional.max_pool1d(w[b, :, :lens[b]].view(Hkv, 2, -1).amax(1)[None], 7, stride=1, padding=3)[0]
                assert torch.equal(idx[l, b, :, :kk].long(), torch.sort(P, dim=-1, descending=True, stable=True)[1][:, :kk]), (l, b)
                assert (idx[l, b, :, kk:] == -1).all()


@pytest.mark.parametrize("n,k", [(60_000_001, 5), (100_000_000, 50)], ids=["60m_k5", "100m_k50"])
def test_selection_of_few_among_tens_of_millions_in_one_bin(rk, n, k):
    """So many positions in the bin of the K-th score that the last part's estimate leaves it no stretch: every rank is written."""
    say("selection, few ranks of one huge bin", n, k)
    w = torch.ones(1, 1, n, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(k)
    at = torch.randperm(n, generator=g, device="cuda")[:k - 2]
    w[0, 0, at] = 1.0 + torch.arange(1, k - 1, device="cuda") * 2.0 ** -10       # ... and two ranks among the equal ones
    geom = rk.Geom(1, 1, 1, 128, SCALE)
    ws = rk.Workspace(geom, n, k)
    lens = torch.tensor([n], dtype=torch.int32, device="cuda")
    idx = torch.full((1, 1, k), -7, dtype=torch.int32, device="cuda")
    sel = torch.full((1, 1, k), -7.0, device="cuda")
    for _ in range(2):
        rk.rk_topk_select(geom, w, lens, n, k, 1, idx, sel_scores=sel, workspace=ws)
    torch.cuda.synchronize()
    taken = set(at.tolist())
    rest = [j for j in range(k + 2) if j not in taken][:2]
    assert idx[0, 0].tolist() == at.flip(0).tolist() + rest
    assert torch.equal(sel[0, 0], w[0, 0, idx[0, 0].long()])


def _us(call, per_graph=10, replays=9):
    """Shortest time of a call inside a captured graph."""
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(stream):
        call()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(per_graph):
                call()
        best = float("inf")
        for _ in range(replays):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            graph.replay()
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 1000 / per_graph)
    return best


# (call, rows, bound far above them, most that it may cost against a bound of the rows themselves: half way between the ratio of a launch whose workgroups
# beyond the rows leave at once, 1.10 / 1.33 / 1.36 / 1.27, and with their scores requested first, 1.71 / 2.05 / 1.87 / 1.75)
LOOSE_BOUNDS = [("topk", 65536, 1 << 20, 1.4), ("weights", 8192, 1 << 19, 1.7), ("scores", 8192, 1 << 19, 1.6), ("refresh", 8192, 1 << 19, 1.5)]


@pytest.mark.parametrize("case", LOOSE_BOUNDS, ids=[c[0] for c in LOOSE_BOUNDS])
def test_bound_far_above_the_length_costs_little(rk, case):
    """max_len bounds seq_lens and no more: a captured step's holds for the whole run.  Nothing between the two is read."""
    what, n, cap, most = case
    say("loose bound", *case[:3])
    Hq, Hkv, k = 32, 8, 1024
    g = torch.Generator(device="cuda").manual_seed(n)
    geom = rk.Geom(1, Hq, Hkv, 128, SCALE)
    lens = torch.tensor([n], dtype=torch.int32, device="cuda")
    idx = torch.zeros(1, Hkv, k, dtype=torch.int32, device="cuda")
    q = torch.randn(1, Hq, 128, generator=g, device="cuda").to(torch.bfloat16)
    out = torch.empty_like(q)
    if what != "topk":
        K = torch.zeros(1, Hkv, cap, 128, dtype=torch.bfloat16, device="cuda")
        K[:, :, :n] = torch.randn(1, Hkv, n, 128, generator=g, device="cuda").to(torch.bfloat16)
    us, found = {}, {}
    for bound in (n, cap):
        ws = rk.Workspace(geom, bound, k)
        w = torch.zeros(1, Hq, bound, device="cuda")
        if what == "topk":
            w[:, :, :n] = torch.rand(1, Hq, n, generator=torch.Generator(device="cuda").manual_seed(1), device="cuda")
            call = lambda: rk.rk_topk_select(geom, w, lens, bound, k, 7, idx, workspace=ws)
        elif what == "weights":
            call = lambda: rk.rk_full_attn(geom, q, K, K, lens, bound, out, weights=w, workspace=ws)
        elif what == "scores":
            call = lambda: rk.rk_score_select(geom, q, K, lens, bound, k, 7, idx, workspace=ws)
        else:
            call = lambda: rk.rk_full_attn_select(geom, q, K, K, lens, bound, out, k, 7, idx, workspace=ws)
        us[bound] = _us(call)
        found[bound] = idx.clone()
    say("  %.2f us, bound of %d: %.2f us, %.2f" % (us[n], cap, us[cap], us[cap] / us[n]))
    if what == "topk":
        assert torch.equal(found[n], found[cap])
    assert us[cap] <= most * us[n]
