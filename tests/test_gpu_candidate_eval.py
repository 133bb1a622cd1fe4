"""The re-evaluation of the compact selection's candidates and the finish over them, at the sizes where their work
splits change: batches of candidates a workgroup holds at a time, every token a candidate, classes of equal votes around
the number the finish ranks at once.  check_compact compares every stage with the oracle and with the five-call form."""
import numpy as np
import pytest

import oracle
import workloads as W
from parity_util import oracle_decode
from test_gpu_compact_selection import check_compact, make_layer, gpu   # noqa: F401  (gpu is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,H_kv,D", [(W.BF16, 32, 8, 128), (W.BF16, 28, 4, 128), (W.BF16, 128, 16, 128),
                                            (W.BF16, 6, 2, 64), (W.F32, 64, 8, 128), (W.F32, 24, 8, 64), (W.BF16, 32, 32, 128)])
def test_short_sequences_whose_tokens_are_all_candidates(gpu, dtype, H, H_kv, D):
    w = W.make_workload("short", dtype=dtype, B=4, H=H, H_kv=H_kv, D=D, seq_lens=[1, 127, 1025, 2049], k=1024, beta=2.5,
                        planted_per_head=0, seed=91)
    layer, q = make_layer(w)
    check_compact(w, layer, q, label="short H%d/%d D%d" % (H, H_kv, D))


@pytest.mark.parametrize("copies", [1, 2, 255, 256, 257, 700])
@pytest.mark.parametrize("k", [1, 500, 2000])
def test_equal_votes_around_the_cut(gpu, copies, k):
    """`copies` tokens share the key row of the token in rank k: their votes are equal bit for bit, and the cut goes
    to the lowest indices among them."""
    w = W.make_workload("ties", dtype=W.BF16, H=8, H_kv=2, D=64, seq_lens=[4500], k=k, beta=2.5, planted_per_head=20, seed=92)
    ora = oracle_decode(w, 0)
    order = np.argsort(-ora["votes"], kind="stable")
    slots = w.slots_of(0)
    rows = w.k_pool.reshape(-1, w.H_kv, w.D)
    rows[slots[order[-copies:]]] = rows[slots[order[k - 1]]]
    layer, q = make_layer(w)
    check_compact(w, layer, q, label="ties %d k %d" % (copies, k))
