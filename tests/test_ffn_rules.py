"""The choice of the kernel family against the tables that the schedule makes (the oracle's, on the host): where the library
says that a product's 128-row tiles are taken in pairs, the pairs are there and save the second of two rounds, or nearly half
of many.  (The library knows
the rows and the experts, not the table: one table in eight may be a tile or two off.)"""
import math

import numpy as np
import pytest

import moe_workloads as W
from oracle import moe_oracle as O
from paper_2506_12417_amd import binding as B
from paper_2506_12417_amd.layer import XCDS, default_q_tokens

GRID = 256                       # compute units
WHOLE = 128 | B.MOE_TILE_WHOLE_PLAN


def table(T, E, k, zipf, rng):
    """The 128-row tile table of T tokens that choose k experts each by Zipf shares."""
    if E == 1:
        counts = np.array([T])
    else:
        share = W.zipf_shares(E, zipf, int(rng.integers(1 << 30)))
        pick = np.argsort(np.log(rng.random((T, E))) / share, axis=1)[:, -k:]
        counts = np.bincount(pick.ravel(), minlength=E)
    S = O.schedule_harmoeny(counts, XCDS, default_q_tokens(B.MOE_BF16))
    return O.tiles_from_schedule(S, np.concatenate([[0], np.cumsum(counts)]), 128)


def paired(tiles):
    n = i = 0
    while i < len(tiles):
        a, b = tiles[i], tiles[min(i + 1, len(tiles) - 1)]
        i += 2 if i + 1 < len(tiles) and a[0] == b[0] and a[2] == 128 and a[1] + a[2] == b[1] else 1
        n += 1
    return n


def rounds(tiles, starts, cb):
    """Rounds of items of the single tiles and of the pairs: by all work-groups or by each bin's, as the launches of one
    round decide (by bins where five eighths of the fullest bin's tiles are one)."""
    per_bin = GRID // XCDS
    bins = [tiles[a:b] for a, b in zip(starts[:-1], starts[1:])]
    most = max(len(t) for t in bins)
    single = min(-(-len(tiles) * cb // GRID), -(-most * cb // per_bin))
    if -(-5 * most // 8) * cb > per_bin:
        return single, -(-paired(tiles) * cb // GRID)
    return single, -(-max(paired(t) for t in bins) * cb // per_bin)


# (experts, choices, the products' terms and weight rows, tokens)
FAMILIES = [(1, 1, [(2048, 11264), (5632, 2048)], (1, 1023)), (128, 1, [(768, 3072), (3072, 768)], (1, 16384)),
            (60, 4, [(2048, 2816), (1408, 2048)], (1, 8192)), (8, 2, [(4096, 28672), (14336, 4096)], (1, 4095)),
            (4, 2, [(2048, 4096), (3072, 2048)], (100, 2040)), (16, 2, [(1536, 2048), (1472, 1536)], (100, 8000)),
            (24, 2, [(2304, 1024), (2048, 1536)], (100, 8192)), (48, 1, [(2304, 768), (4096, 512)], (100, 32000))]


@pytest.mark.parametrize("E,k,products,tokens", FAMILIES)
def test_pairs_are_taken_only_where_they_save_rounds(E, k, products, tokens):
    rng, said, wrong = np.random.default_rng(E), 0, []
    for _ in range(300):
        T = int(round(math.exp(rng.uniform(math.log(tokens[0]), math.log(tokens[1])))))
        if not any(B.moe_ffn_pairs(WHOLE, T * k, E, K, N) for K, N in products):
            continue
        tiles, starts = table(T, E, k, rng.uniform(0, 2.0 if E == 8 else 1.5), rng)
        for K, N in products:
            cb = (N + 255) // 256
            if B.moe_ffn_pairs(WHOLE, T * k, E, K, N):
                said += 1
                single, pairs = rounds(tiles, starts, cb)
                if not (single >= 2 and pairs == 1 or K >= 4096 and pairs >= 8 and paired(tiles) <= 0.6 * len(tiles)):
                    wrong.append((T, K, N, rounds(tiles, starts, cb)))
    assert said >= 5 or E in (60, 128)
    assert len(wrong) <= said // 8, wrong


def test_nothing_is_paired_where_every_expert_has_one_tile_or_the_items_fit_one_round():
    for A in range(1, 641):
        assert not B.moe_ffn_pairs(WHOLE, A, 1, 2048, 11264) and not B.moe_ffn_pairs(WHOLE, A, 1, 5632, 2048), A
    for T in range(1, 400):
        assert not B.moe_ffn_pairs(WHOLE, 4 * T, 60, 1408, 2048), T
    for T in range(1, 16385, 7):
        assert not B.moe_ffn_pairs(WHOLE, T, 128, 3072, 768), T
    assert not B.moe_ffn_pairs(WHOLE, 1792, 24, 2560, 2560)
    assert B.moe_ffn_pairs(WHOLE, 768, 1, 2048, 11264) and B.moe_ffn_pairs(WHOLE, 1023, 1, 2048, 11264)


def test_a_plan_over_some_of_the_experts_is_never_paired():
    """A call that does not say that its plan covers all rows (a group of experts, moe_plan_tiles_subset) cannot be judged by them."""
    for A in range(64, 32769, 64):
        for E in (1, 8, 32):
            for K, N in ((2048, 11264), (3072, 768), (14336, 4096)):
                assert not B.moe_ffn_pairs(128, A, E, K, N) and not B.moe_ffn_pairs(256 | B.MOE_TILE_WHOLE_PLAN, A, E, K, N)
    assert B.moe_ffn_pairs(WHOLE, 12000, 32, 3072, 768)
