"""Which form of the selection a decode step takes (host rule).  Above 24 MiB of score matrices the candidates are ranked by votes
of double-precision products whatever k, the heads and the batch are; below, one sequence is from where that was the faster form
when the line was laid (it has become faster since, and the line stays: the votes that rank a call change with the form)."""
from types import SimpleNamespace

import pytest

pytest.importorskip("torch")
from paper_2411_02886_amd.runtime import DecodeLayer


@pytest.mark.parametrize("B,n,H,D,k,compact", [
    (1, 131072, 32, 128, 2048, False),      # 16 MiB
    (1, 139264, 32, 128, 2048, False),      # 17 MiB: 92 us, compact 95
    (1, 69632, 64, 128, 2048, False),       # 17 MiB: 68 us, compact 72
    (1, 159744, 32, 128, 2048, False),      # 19.5 MiB: 102 us, compact 97
    (1, 163840, 32, 128, 2048, True),       # 20 MiB: 107 us, compact 97
    (1, 97894, 64, 128, 2048, False),       # 23.9 MiB: 83 us, compact 77
    (2, 98304, 32, 128, 2048, False),       # 24 MiB, the line of a batch itself
    (2, 98305, 32, 128, 2048, True),
    (1, 98305, 64, 128, 2048, True),
    (1, 1048576, 28, 128, 4096, True),
    (1, 4096, 8, 64, 256, False),
    (32, 16001, 32, 128, 2048, True),       # 62.5 MiB: short sequences with a large k, too
    (32, 16001, 32, 128, 256, True),
    (32, 8180, 64, 128, 2154, True),
    (4, 40009, 64, 128, 2048, True),
    (8, 65536, 32, 128, 2048, True),
    (4, 198163, 32, 64, 2195, True),
    (16, 500, 128, 128, 1 << 20, False),
])
def test_form(B, n, H, D, k, compact):
    assert DecodeLayer.compact_form_pays(SimpleNamespace(B=B, max_seq_len=n, H=H, D=D, k=k)) is compact
