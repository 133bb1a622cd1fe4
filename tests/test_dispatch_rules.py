"""Host rules that choose between kernels and split their work, checked without a GPU."""
import random

import numpy as np
import pytest

from rules_util import MASKED, WHOLE, rules, score_shape, score_share


def test_streaming_attention_splits_are_legal_and_fit_the_workspace():
    L, rng = rules(), random.Random(1)
    for _ in range(20000):
        pairs, total = rng.choice([rng.randint(1, 64), rng.randint(1, 65535 * 32)]), rng.randint(1, 32768)
        chunks = (total + 63) // 64                    # what the workspace holds partials for
        if chunks * pairs < 1024:                      # never streamed
            continue
        span = L.rule_stream_span(pairs, total)
        assert 32 <= span <= 3584 and span % 32 == 0, (pairs, total, span)
        assert (total + span - 1) // span <= chunks, (pairs, total, span)


@pytest.mark.parametrize("total", [2048, 2688, 4096, 4736])
def test_streaming_attention_splits_fill_the_rounds(total):
    """A last round that a few workgroups have to themselves costs as much as a full one: 96 pairs in three runs each are
    288 workgroups, two rounds of which one is an eighth full."""
    L = rules()
    for pairs in range(48, 700):
        span = L.rule_stream_span(pairs, total)
        runs = (total + span - 1) // span
        rounds = (pairs * runs + 255) // 256
        whole = pairs * total / 256                    # keys per CU if nothing were left over
        # 1.5: 171 pairs in one run each, a third of the CUs without work, where two runs and their merge cost more
        assert rounds * span <= 1.5 * whole + 160, (pairs, runs)


@pytest.mark.parametrize("G,D,pairs,total,streamed", [
    # measured, us in 64-token chunks and streamed
    (1, 64, 144, 2048, 0), (1, 64, 288, 2048, 0), (1, 64, 384, 2048, 0),       # 20.2 / 22.4, 35.2 / 37.5, 43 / 44
    (1, 128, 144, 2048, 0), (1, 128, 112, 4096, 0),                            # 30.1 / 33.7, 42 / 47
    (2, 64, 288, 2048, 0), (2, 64, 384, 2048, 0), (2, 128, 136, 4000, 0),      # 35.6 / 36.9, 43 / 45, 53 / 55
    (1, 64, 720, 2048, 1), (1, 128, 368, 2048, 1), (2, 128, 368, 2048, 1),     # 80 / 75, 81 / 71, 85 / 72
    (1, 64, 832, 300, 1), (1, 128, 480, 700, 1), (1, 128, 528, 700, 0),        # 20 / 16, 35 / 33, 39 / 44
    (2, 64, 648, 700, 1), (2, 128, 424, 700, 1),                               # 31 / 27, 36 / 30
    (4, 128, 64, 2048, 1), (3, 64, 128, 1000, 1), (8, 128, 64, 1000, 1)])      # 21.8 / 18.1, 15.1 / 13.2, 20.9 / 13.2
def test_streaming_attention_only_where_it_is_the_faster_form(G, D, pairs, total, streamed):
    assert rules().rule_attn_streams(G, D, pairs, total) == streamed


@pytest.mark.parametrize("batch", [1, 2, 3, 8, 100, 171, 200, 300, 511, 600])
@pytest.mark.parametrize("k", [1, 64, 4096])
def test_candidates_are_evaluated_by_a_full_chip_whatever_k(batch, k):
    """With flat votes every token is a candidate: the workgroups are counted by what a sequence can hold, not by k."""
    for n in (1, 4, 5, 1000, 2048, 131072, 1 << 20):
        parts = rules().rule_eval_workgroups(batch, n, k)
        assert 1 <= parts <= 512
        assert parts <= (n + 3) // 4                      # four candidates each, at least
        if n >= 2048:                                     # 512 workgroups a round, the rounds at least two thirds full
            assert batch * parts >= 341 * ((batch * parts + 511) // 512), (batch, n)


@pytest.mark.parametrize("G,D,pairs,total,streamed", [
    # three heads and more, us in chunks and streamed: lists of one run ...
    (4, 64, 2, 256, 1), (4, 64, 2, 300, 1), (3, 64, 1, 257, 1), (6, 128, 2, 16, 1), (8, 128, 168, 748, 1), (3, 64, 120, 287, 1), (4, 128, 64, 277, 1),
    # ... and the two sides of the lines with splits
    (4, 64, 2, 352, 0), (8, 128, 1, 352, 0), (8, 128, 8, 1429, 0), (8, 128, 24, 915, 1), (7, 128, 8, 2228, 0), (7, 128, 40, 679, 1), (5, 128, 8, 3072, 0), (5, 128, 48, 1565, 1),
    (4, 128, 16, 1291, 0), (4, 128, 24, 3385, 1), (4, 64, 24, 3055, 0), (4, 64, 16, 5637, 1), (3, 64, 24, 3636, 0), (3, 64, 104, 960, 1)])
def test_short_calls_stream_from_their_own_lines_on(G, D, pairs, total, streamed):
    assert rules().rule_attn_streams(G, D, pairs, total) == streamed


def test_every_streamed_call_has_room_for_its_splits():
    L, rng = rules(), random.Random(2)
    for _ in range(20000):
        G, D, pairs, total = rng.randint(3, 8), rng.choice([64, 128]), rng.randint(1, 64), rng.choice([rng.randint(1, 400), rng.randint(1, 32768)])
        if not L.rule_attn_streams(G, D, pairs, total):
            continue
        span = L.rule_stream_span(pairs, total)
        assert 32 <= span <= 3584 and span % 32 == 0, (pairs, total, span)
        assert (total + span - 1) // span <= (total + 63) // 64, (pairs, total, span)


def test_flat_votes_scratch_fits_the_lists_memory():
    for batch in (1, 2, 7, 300, 65535):
        for n in (1, 2048, 2049, 8193, 1048576, 1048577):
            assert rules().rule_topk_scratch_fits(batch, n), (batch, n)


def test_units_of_the_shared_score_grid_are_divided_exactly():
    """Runs of 1, 2, 4, 6 and 8 tiles for one, two and four waves; tiles of up to 2^31 tokens."""
    L, rng = rules(), random.Random(3)
    for d in sorted({g * r for g in (1, 2, 4) for r in (1, 2, 4, 6, 8)}):
        most = 2**26 + d
        xs = list(range(0, 5 * d)) + [rng.randrange(most) for _ in range(2000)] + [most - i for i in range(3 * d)]
        xs += [q * d + e for q in (rng.randrange(most // d) for _ in range(500)) for e in (0, d - 1)]
        for x in xs:
            assert L.rule_unit_div(x, d) == x // d, (x, d)


def check_share(B, H, H_kv, D, max_len, dense, lens, skip):
    """Every tile of every scanned sequence belongs to one wave of each slice of the KV heads, the workgroups fit the grid and the
    partials' section, the runs of a masked call their LDS; returns the units of a workgroup over the fewest it could take."""
    case = (B, H, H_kv, D, max_len, dense, lens, skip)
    shape = score_shape(B, H, H_kv, D, max_len, dense, WHOLE if skip is None else MASKED)
    groups = 4 // shape.NU
    assert shape.lds <= 163840 and shape.lds * (shape.grid // 256) <= 163840, case
    rows = score_share(B, H, H_kv, D, max_len, dense, lens, skip)
    wg, wave, b, x, n, base, tiles, uw = rows.T
    for s in range(B):
        mine = b == s
        if skip is not None and skip[s]:
            assert not mine.any(), case
            continue
        ntt = (lens[s] + 31) // 32
        cnt = int(n[mine][0])
        assert sorted(set(wg[mine])) == list(range(wg[mine].min(), wg[mine].min() + cnt)), case      # none cut off by the grid
        assert sorted(set(x[mine])) == list(range(cnt)) and cnt <= 1024, case
        for u in range(shape.NU):
            sel = mine & (wave % shape.NU == u)
            edges = sorted((f, f + t) for f, t in zip(base[sel], tiles[sel]) if t > 0)
            assert [f for f, _ in edges] == [0] * bool(edges) + [e for _, e in edges[:-1]] and (edges[-1][1] if edges else 0) == ntt, case
        if skip is not None:
            runs = -(-ntt // shape.SR)
            assert max(1, -(-runs // groups)) <= 1024 and uw.max() * groups * H * 8 <= shape.run_stat_bytes, case
            part = wave[mine] // shape.NU
            live = tiles[mine] > 0
            assert (base[mine][live] == ((x[mine] * uw[mine] * groups + part * uw[mine]) * shape.SR)[live]).all(), case
            assert (tiles[mine] <= uw[mine] * shape.SR).all(), case
    return int(uw[0]) // (groups if skip is None else 1)


_SCORE_HEADS = [(24, 8), (32, 8), (28, 4), (32, 4), (40, 8), (64, 8), (48, 16), (64, 16), (96, 32), (128, 32), (80, 16), (128, 16)]


def test_a_shared_score_grid_covers_every_tile_once():
    rng, seen = random.Random(4), set()
    for i in range(700):
        (H, H_kv), D, dense, masked = rng.choice(_SCORE_HEADS), rng.choice([64, 128]), rng.random() < 0.5, rng.random() < 0.5
        B = rng.choice([2, 3, 5, 8, 16, 33, 63, 64])
        longest = int(2 ** rng.uniform(6, 19 - np.log2(B) / 2))
        lens = [rng.choice([rng.randint(0, longest), longest, rng.randint(0, 70), rng.randint(longest // 2, longest)]) for _ in range(B)]
        lens = [min(n, longest) for n in lens]
        shape = score_shape(B, H, H_kv, D, longest, dense, MASKED if masked else WHOLE)
        if shape is None or not shape.shared:
            continue
        skip = [int(rng.random() < 0.4) for _ in range(B)] if masked else None
        if masked and all(skip):
            skip[0] = 0
        units = check_share(B, H, H_kv, D, longest, dense, lens, skip)
        seen.add((masked, shape.NU, units > 1))
    assert seen == {(m, nu, more) for m in (False, True) for nu in (1, 2, 4) for more in (False, True)}


def test_the_runs_of_a_masked_score_grid_are_those_of_a_call_alone():
    """The bits of a sequence's statistics: one run of SR tiles per wave, as a launch of the sequence by itself has them."""
    rng, n = random.Random(5), 0
    for _ in range(3000):
        (H, H_kv), D, dense = rng.choice(_SCORE_HEADS), rng.choice([64, 128]), rng.random() < 0.5
        B, longest = rng.randint(2, 64), int(2 ** rng.uniform(8, 19))
        shape = score_shape(B, H, H_kv, D, longest, dense, MASKED)
        if shape is None or not shape.shared:
            continue
        alone = score_shape(1, H, H_kv, D, longest, dense, WHOLE)
        assert alone is not None and not alone.shared and alone.RR == shape.SR, (B, H, H_kv, D, longest, dense)
        assert alone.grid < 1024 and alone.grid * 4 >= -(-((longest + 31) // 32) // alone.RR) * alone.NU      # one run per wave
        n += 1
    assert n > 300


@pytest.mark.parametrize("H,H_kv", [(40, 8), (48, 8), (56, 8), (80, 16), (112, 16)])
def test_masked_score_matrices_that_leave_in_pieces_do_not_share_the_grid(H, H_kv):
    """40/8, D 64, 8 x 40960 tokens, all of them: 88 us shared, 76 in a grid of their own; their bytes 58 and 70."""
    for D in (64, 128):
        longest = 40960 * 8 * 64 // (H_kv * D)
        assert not score_shape(8, H, H_kv, D, longest, True, MASKED).shared
        assert score_shape(8, H, H_kv, D, longest, False, MASKED).shared
    assert score_shape(8, 28, 4, 128, 10240, True, MASKED).shared and score_shape(8, 64, 8, 64, 20480, True, MASKED).shared
