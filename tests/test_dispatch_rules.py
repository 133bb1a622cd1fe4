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
