"""The ranked vote where its workgroup changes: 512 threads over 256 tokens or 1024 over 512 (16 and 17 heads; 17 to 32 heads at
128 and 256 large workgroups), lengths at, before and past a workgroup's last token, one, two and four pieces per lane."""
import pytest

import workloads as W
from test_gpu_decode_parity import gpu  # noqa: F401  (a fixture)
from test_gpu_ranked_vote import test_ranked_pair_agrees_with_the_plain_pair_and_restores_the_workspace as check

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(W.F32, 16, 4, 64, [8449, 8448, 8447]), (W.F32, 20, 4, 64, [8449, 8448, 255, 257]),
                                   (W.BF16, 24, 8, 64, [65536]), (W.BF16, 24, 8, 64, [65537]),
                                   (W.BF16, 24, 8, 64, [131072]), (W.BF16, 24, 8, 64, [131073]), (W.BF16, 40, 8, 64, [8705, 3]),
                                   (W.BF16, 128, 16, 64, [8704, 256])], ids=lambda s: "dt%d_H%d_%d_D%d_%s" % s)
def test_workgroup_edges(gpu, shape):
    check(gpu, shape, (0, 0))
