"""Which form of the selection a decode step takes (host rule): the sides of both lines, and the sizes it was measured at."""
from types import SimpleNamespace

import pytest

pytest.importorskip("torch")
from paper_2411_02886_amd.runtime import DecodeLayer


@pytest.mark.parametrize("B,n,H,D,k,compact", [
    (1, 131072, 32, 128, 2048, False),      # 16 MiB
    (1, 163711, 28, 128, 903, True),        # 17.5 MiB in one sequence
    (1, 1048576, 28, 128, 4096, True),
    (1, 4096, 8, 64, 256, False),
    (32, 16001, 32, 128, 2048, False),      # 62.5 MiB, 268 million products
    (32, 16001, 32, 128, 256, True),        # the same with 34 million
    (4, 198163, 32, 64, 2195, True),
    (16, 500, 128, 128, 1 << 20, False),    # k beyond the sequence counts as the sequence
])
def test_form(B, n, H, D, k, compact):
    assert DecodeLayer.compact_form_pays(SimpleNamespace(B=B, max_seq_len=n, H=H, D=D, k=k)) is compact
