"""Chunked-prefill selection where the chunk's rows (queries x query heads of a KV head) end inside a workgroup's 256: waves without a
row only stage K, waves with one row to 64."""
import pytest

import workloads as W
from test_gpu_prefill_parity import check_chunk, gpu   # noqa: F401  (gpu is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("C,H,H_kv,D", [(64, 8, 8, 64), (65, 8, 8, 128), (128, 4, 4, 64), (43, 6, 2, 128), (193, 2, 2, 64), (257, 2, 2, 128), (46, 28, 4, 64)])
def test_rows_that_end_inside_a_workgroup(gpu, C, H, H_kv, D):
    w = W.make_workload("rows", dtype=W.BF16, B=2, C=C, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[C + 700, C + 65], k=80, seed=C + H, beta=2.5,
                        planted_per_head=3)
    print("rows", C * H // H_kv, flush=True)
    check_chunk(gpu, w, 80, 0.2, "rows %d" % (C * H // H_kv))
