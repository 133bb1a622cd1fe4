"""The passes over all votes of ts_topk (flat votes): the threshold's last ten key bits at both ends of their range and between,
ties that begin, end and are cut at the edges of the 2048-token chunks, and both sides of the length from which a counting
pass takes the table's place.  Every selection is compared with a stable sort; the calls share a workspace."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _layer(lens, k, num_initial=0, num_local=0):
    from paper_2411_02886_amd.runtime import DecodeLayer
    pages = [(n + 15) // 16 for n in lens]
    indptr = np.concatenate([[0], np.cumsum(pages)]).astype(np.int32)
    pool = torch.zeros((1, 16, 1, 64), dtype=torch.int16, device="cuda:0")      # ts_topk looks at the votes only
    return DecodeLayer(H=1, H_kv=1, D=64, P=16, k=k, dtype=1, k_pool=pool, v_pool=pool, page_indptr=indptr,
                       page_indices=np.zeros(int(indptr[-1]), np.int32), seq_lens=np.array(lens, np.int32),
                       num_initial=num_initial, num_local=num_local)


def _votes(kind, n, rng):
    one = np.float32(1.0).view(np.uint32)
    if kind == "spread":
        return rng.random(n).astype(np.float32)
    if kind == "equal":
        return np.full(n, 0.5, np.float32)
    if kind == "last digit":            # the upper 22 bits the same for most: every value of the last digit
        v = (one + rng.integers(0, 1024, n).astype(np.uint32)).view(np.float32).copy()
        v[rng.integers(0, n, max(1, n // 3000))] = 3.0
        return v
    if kind == "top of the digit":      # the threshold is the digit's largest value, ties in long runs
        v = (one + np.uint32(1023) * (np.arange(n) // 1500 % 2).astype(np.uint32)).view(np.float32).copy()
        v[rng.integers(0, n, max(1, n // 5000))] = 2.0
        return v
    raise ValueError(kind)


def _check(layer, lens, k, votes, lo=0, tail=0):
    import paper_2411_02886_amd as ts
    from paper_2411_02886_amd.runtime import to_host
    for b, v in enumerate(votes):
        layer.votes[b, :len(v)] = torch.from_numpy(v).to("cuda:0")
    layer.idx.fill_(-7); layer.count.fill_(-7)
    ts.ts_topk(layer.problem, layer.votes, k, layer.idx, layer.count, None, layer.ws, flags=ts.TS_TOPK_FLAT_VOTES)
    torch.cuda.synchronize()
    idx, count = to_host(layer.idx), to_host(layer.count)
    for b, n in enumerate(lens):
        a = min(lo, n)
        e = max(a, n - tail)
        order = np.argsort(-votes[b][a:e].astype(np.float64), kind="stable")[:k]
        want = np.sort(order) + a
        assert count[b] == len(want), b
        assert np.array_equal(idx[b, :len(want)], want), b
        assert (idx[b, len(want):] == -1).all(), b


KINDS = ["spread", "equal", "last digit", "top of the digit"]


@pytest.mark.parametrize("lens,lo,tail", [([8193], 0, 0), ([20000, 0, 2048, 2049], 0, 0), ([12288, 4095, 1], 100, 61), ([1048576], 0, 0), ([1048577, 5], 0, 0)])
@pytest.mark.parametrize("k", [1, 300, 2049, 8192])
def test_flat_votes_against_a_stable_sort(lens, lo, tail, k):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("flat topk", lens, lo, tail, k, flush=True)
    rng = np.random.default_rng(len(lens) * 100000 + k)
    layer = _layer(lens, k, lo, tail)
    for kind in KINDS + KINDS[:2]:
        _check(layer, lens, k, [_votes(kind, n, rng) if n else np.zeros(0, np.float32) for n in lens], lo, tail)


def test_lengths_on_both_sides_of_the_line_share_a_workspace():
    """The histograms that a call leaves serve the next one, whichever of the two ways either takes."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(7)
    long, short = _layer([1048577], 500), _layer([30000], 500)
    short.ws = long.ws                                   # sized for the longer sequence
    import paper_2411_02886_amd as ts
    ts.ts_workspace_init(long.ws)
    for kind in ["last digit", "spread", "equal", "top of the digit"]:
        for layer, n in ((long, 1048577), (short, 30000), (short, 30000), (long, 1048577)):
            print("shared workspace", kind, n, flush=True)
            _check(layer, [n], 500, [_votes(kind, n, rng)])


@pytest.mark.parametrize("lens", [[20000, 0, 9000], [1048576], [1048577, 5]])
def test_histograms_are_zero_again_after_the_call(lens):
    """All of the workspace up to its state words: a call for a smaller batch has other histograms there."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from rules_util import rules
    print("zero again", lens, flush=True)
    rng = np.random.default_rng(11)
    layer = _layer(lens, 300)
    for kind in KINDS:
        _check(layer, lens, 300, [_votes(kind, n, rng) if n else np.zeros(0, np.float32) for n in lens])
        zeroed = layer.ws[:rules().rule_zeroed_bytes(len(lens), max(lens)) // 4]
        assert zeroed.numel() >= len(lens) * 10 * 2048 and not zeroed.any(), kind


@pytest.mark.parametrize("n,H,H_kv", [(8256, 32, 8), (8257, 32, 8), (8257, 16, 8), (20001, 28, 4)])
def test_mean_query_selection_with_and_without_the_vote_launch_histogram(n, H, H_kv):
    """select_mean_query on either side of its line, twice in a row, against the plain pair of calls on the same scores."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02886_amd as ts
    import workloads as W
    from paper_2411_02886_amd.runtime import ChunkSelector, to_device
    print("mean query", n, H, flush=True)
    w = W.make_workload("mq", dtype=W.BF16, B=2, C=64, H=H, H_kv=H_kv, D=64, P=16, seq_lens=[n, 5000], k=300, seed=n + H)
    sel = ChunkSelector.from_workload(w)
    q = to_device(w.q)
    got = []
    for _ in range(2):
        sel.idx.fill_(-7); sel.votes.fill_(-1.0)
        sel.select_mean_query(q, 1.0)
        got.append((sel.idx.clone(), sel.votes.clone(), sel.count.clone()))
    m = sel._mq
    ts.ts_paged_qk_scores(m["problem"], m["q_mean"], m["scores"], 1.0, None, m["ws"])
    sel.votes.fill_(-1.0)
    ts.ts_soft_vote(m["problem"], m["scores"], 1.0, m["row_stats"], sel.votes, None, m["ws"])
    ts.ts_topk(m["problem"], sel.votes, sel.k, sel.idx, sel.count, None, m["ws"])
    torch.cuda.synchronize()
    for idx, votes, count in got:
        assert torch.equal(idx, sel.idx) and torch.equal(votes, sel.votes) and torch.equal(count, sel.count)
