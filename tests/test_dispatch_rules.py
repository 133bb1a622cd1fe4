"""Host rules that choose between kernels and split their work, checked without a GPU."""
import random

import pytest

from rules_util import rules


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
