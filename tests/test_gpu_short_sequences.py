"""Short sequences: the TopK by one workgroup per sequence around the sizes where its votes per thread change, and the
ranked vote that merges the score pass's statistics itself, also with more of them than its launch expects."""
import numpy as np
import pytest

import oracle
import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02886_amd as ts
    ts.load()
    return ts


@pytest.mark.parametrize("longest", [1, 63, 4095, 4096, 4097, 8191, 8192, 8193, 16385])
@pytest.mark.parametrize("kind", ["spread", "flat", "ties", "signed"])
def test_topk(gpu, longest, kind):
    from paper_2411_02886_amd import binding as ts
    rng = np.random.default_rng(longest)
    B, ni, nl = 3, 5, 7
    lens = np.array([longest, max(1, longest // 2), 0], np.int32)
    votes = {"spread": np.exp(rng.standard_normal((B, longest)) * 6), "flat": 1 + rng.random((B, longest)) * 1e-3,
             "ties": rng.integers(0, 4, (B, longest)).astype(np.float64), "signed": rng.standard_normal((B, longest))}[kind].astype(np.float32)
    dev = "cuda:0"
    seq = torch.from_numpy(lens).to(dev)
    dummy = torch.zeros(64, dtype=torch.int32, device=dev)
    v = torch.from_numpy(votes).to(dev)
    for k in (1, 100, 5000):
        p = ts.Problem(batch=B, num_q_heads=8, num_kv_heads=2, head_dim=64, page_size=16, max_seq_len=longest, dtype=ts.TS_F32,
                       k_pool=v, v_pool=v, page_indptr=dummy, page_indices=dummy, seq_lens=seq, num_initial=ni, num_local=nl)
        ws = torch.empty((ts.ts_workspace_bytes(p, k) + 255) // 256 * 64, dtype=torch.int32, device=dev)
        ts.ts_workspace_init(ws)
        print("short topk", longest, kind, k, flush=True)
        for flags in (0, ts.TS_TOPK_FLAT_VOTES):
            idx = torch.full((B, k), -7, dtype=torch.int32, device=dev)
            count = torch.full((B,), -7, dtype=torch.int32, device=dev)
            for again in range(2):
                ts.ts_topk(p, v, k, idx, count, None, ws, flags=flags)
            got_i, got_c = idx.cpu().numpy(), count.cpu().numpy()
            for b in range(B):
                lo, hi = oracle.ranked_range(int(lens[b]), ni, nl)
                order = lo + np.argsort(-votes[b, lo:hi].astype(np.float64), kind="stable")[:k]
                assert got_c[b] == len(order), (b, flags)
                assert np.array_equal(got_i[b, :len(order)], np.sort(order)) and np.all(got_i[b, len(order):] == -1), (b, flags)


@pytest.mark.parametrize("H,H_kv,dtype,lens", [(8, 2, W.F32, [4096, 1, 0]), (32, 8, W.BF16, [4096, 33]), (32, 8, W.BF16, [16384]),
                                               (32, 8, W.BF16, [16500, 900]), (128, 16, W.BF16, [1000]), (6, 2, W.F32, [700])])
@pytest.mark.parametrize("wg", [0, 1, 300, 1024])
def test_ranked_vote_merges_its_statistics(gpu, H, H_kv, dtype, lens, wg):
    """`wg` workgroups in the score pass (0: as it likes), then the votes with the knob back at its default."""
    from paper_2411_02886_amd import binding as ts
    from paper_2411_02886_amd.runtime import DecodeLayer, to_device
    w = W.make_workload("short", dtype=dtype, B=len(lens), H=H, H_kv=H_kv, D=64, seq_lens=lens, k=64, beta=2.5,
                        planted_per_head=0, seed=H + len(lens))
    layer, q = DecodeLayer.from_workload(w), to_device(w.q)
    print("ranked vote", H, H_kv, lens, wg, flush=True)
    got = []
    for ranked in (False, True):
        ts.ts_debug_set_score_variant(2, wg)
        ts.ts_paged_qk_scores(layer.problem, q, layer.scores, 1.0, None, layer.ws)
        ts.ts_debug_set_score_variant(2, 0)
        layer.row_stats.fill_(7.0)
        layer.votes.zero_()
        if ranked:
            ts.ts_soft_vote_ranked(layer.problem, layer.scores, 1.0, layer.row_stats, layer.votes, None, layer.ws)
            ts.ts_topk(layer.problem, layer.votes, layer.k, layer.idx, layer.count, None, layer.ws, flags=ts.TS_TOPK_VOTE_HIST)
        else:
            ts.ts_soft_vote(layer.problem, layer.scores, 1.0, layer.row_stats, layer.votes, None, layer.ws)
            ts.ts_topk(layer.problem, layer.votes, layer.k, layer.idx, layer.count, None, layer.ws)
        got.append([t.clone() for t in (layer.row_stats, layer.votes, layer.idx, layer.count)])
    for plain, ranked in zip(*got):
        assert torch.equal(plain, ranked)
