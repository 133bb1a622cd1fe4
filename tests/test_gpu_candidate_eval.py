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


@pytest.mark.parametrize("dtype,H,H_kv,D", [(W.BF16, 1, 1, 128), (W.BF16, 5, 1, 64), (W.F32, 4, 1, 128), (W.BF16, 6, 2, 128), (W.F32, 16, 2, 64),
                                            (W.BF16, 12, 4, 64), (W.F32, 28, 4, 128), (W.BF16, 64, 8, 128), (W.BF16, 64, 16, 64),
                                            (W.F32, 64, 32, 64), (W.BF16, 128, 16, 128), (W.BF16, 128, 32, 128)])
def test_votes_of_the_candidates_against_64_bits(gpu, dtype, H, H_kv, D):
    """Every number of KV heads and head sets that a wave step is laid out for, with fewer candidates than a step, a step's and
    more: sel_votes against Eq. 5 in 64 bits from the GPU's own statistics.  The products are exact in both; a weight's power of
    two comes from the float exponential (1 ulp, 1.2e-7) of an argument rounded to float (0.5 * 6e-8 * ln 2), the vote is
    rounded once (6e-8): below 3e-7, 5e-7 asserted."""
    from paper_2411_02886_amd.runtime import to_host
    lens, scale = [1, 3, 17, 70, 2500], 0.5
    w = W.make_workload("sel_votes", dtype=dtype, B=len(lens), H=H, H_kv=H_kv, D=D, seq_lens=lens, k=300, beta=2.5, planted_per_head=0, seed=93)
    layer, q = make_layer(w)
    print("candidates' votes", dtype, H, H_kv, D, flush=True)
    layer.select_compact(q, scale, None)
    torch.cuda.synchronize()
    idx, cnt, st, got = (to_host(x) for x in (layer.idx, layer.count, layer.row_stats, layer.sel_votes))
    qf = W.as_f32(w.q, dtype).astype(np.float64)
    rows = W.as_f32(w.k_pool.reshape(-1, H_kv, D), dtype).astype(np.float64)
    for b, n in enumerate(lens):
        m = int(cnt[b])
        assert m == min(n, 300)
        k = rows[w.slots_of(b)[idx[b, :m]]]                                  # [m][H_kv][D]
        s = np.einsum("mhd,hd->mh", np.repeat(k, H // H_kv, axis=1), qf[b, 0])
        ref = (np.exp(float(np.float32(scale)) * (s - st[b, :, 0].astype(np.float64))) / st[b, :, 1].astype(np.float64)).sum(axis=1)
        np.testing.assert_allclose(got[b, :m], ref, rtol=5e-7, err_msg="b %d" % b)


@pytest.mark.parametrize("lens,k", [([200000], 64), ([3, 0, 9000], 2048), ([2500] * 70, 300)])
def test_the_histogram_is_left_zeroed(gpu, lens, k):
    """Every workgroup clears its share of the lower bounds' histogram, with candidates (behind the loads of their rows) or without."""
    from rules_util import rules
    w = W.make_workload("cleared", dtype=W.BF16, B=len(lens), H=8, H_kv=2, D=64, seq_lens=lens, k=k, beta=2.5, planted_per_head=2, seed=94)
    layer, q = make_layer(w)
    for _ in range(2):
        layer.select_compact(q, 1.0, None)
        torch.cuda.synchronize()
        assert not layer.ws[:rules().rule_zeroed_bytes(len(lens), max(lens)) // 4].any()


@pytest.mark.parametrize("dtype,H_kv,D", [(W.BF16, 1, 64), (W.F32, 2, 64), (W.F32, 4, 128), (W.BF16, 8, 128), (W.F32, 8, 128), (W.BF16, 16, 64),
                                          (W.F32, 32, 64), (W.BF16, 32, 128)])
def test_one_query_head_per_kv_head(gpu, dtype, H_kv, D):
    """Products by vector instructions: every number of KV heads, four and eight waves."""
    test_votes_of_the_candidates_against_64_bits(gpu, dtype, H_kv, H_kv, D)


@pytest.mark.parametrize("k,copies", [(1, 1), (7, 5), (1000, 110), (1000, 126), (1000, 400), (4096, 512), (4096, 2500)])
def test_candidates_beyond_those_that_are_loaded_early(gpu, k, copies):
    """The finish asks for k + k / 8 candidates before it knows how many there are: with as many equal votes at the cut there are fewer,
    just as many, and more."""
    w = W.make_workload("early", dtype=W.BF16, H=8, H_kv=2, D=64, seq_lens=[9000], k=k, beta=2.5, planted_per_head=20, seed=95)
    ora = oracle_decode(w, 0)
    order = np.argsort(-ora["votes"], kind="stable")
    slots, rows = w.slots_of(0), w.k_pool.reshape(-1, w.H_kv, w.D)
    rows[slots[order[k - 1:k - 1 + copies]]] = rows[slots[order[k - 1]]]
    layer, q = make_layer(w)
    check_compact(w, layer, q, label="early k %d copies %d" % (k, copies))
