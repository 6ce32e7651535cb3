"""Sizes at which a kernel's tiles, rounds and dispatch rules change hands, against the CPU oracle."""
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


# 64 rows per wavefront, 512 per workgroup and round; 128 pairs leave a pair 4 workgroups (2048 rows per
# round), 520 pairs one; 16 blocks of columns, and a negative scale
WINDOW_EDGES = [("rows_63_64_65", 3, 8, 2, [63, 64, 65], 5, SCALE), ("rows_511_512_513", 3, 4, 4, [511, 512, 513], 32, SCALE),
                ("rows_575_576_577_w1", 3, 8, 1, [575, 576, 577], 1, SCALE), ("three_rounds", 65, 8, 8, [1100, 1025] + [40] * 63, 3, SCALE),
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
