"""The matrix-core score pass for five to eight query heads over 8 and 16 KV heads (two and four wave tiles side by side): both
forms against the oracle, and its scores' error against 64 bits beside the vector kernel's."""
import numpy as np
import pytest

import oracle
import workloads as W
from test_gpu_compact_selection import check_compact, make_layer, gpu   # noqa: F401  (gpu is a fixture)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,H_kv,D,P,lens,k", [
    (64, 8, 128, 16, [1], 4), (64, 8, 128, 1, [31, 33], 20), (40, 8, 128, 2, [2049], 100), (48, 8, 64, 16, [900, 0, 4100], 64),
    (56, 8, 128, 16, [5003], 300), (80, 16, 128, 16, [1300, 65], 50), (112, 16, 64, 1, [700], 40), (128, 16, 128, 4, [2500], 128)])
def test_five_to_eight_heads_over_more_kv_heads(gpu, H, H_kv, D, P, lens, k):
    w = W.make_workload("wide", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=P, B=len(lens), seq_lens=lens, k=k, beta=2.5, planted_per_head=0, seed=H + D + k)
    for ni, nl in ((0, 0), (4, 61)):
        layer, q = make_layer(w, num_initial=ni, num_local=nl)
        print("matrix-core scores", H, H_kv, D, P, lens, ni, nl, flush=True)
        check_compact(w, layer, q, score_scale=1.0, label="wide %d/%d" % (H, H_kv))


@pytest.mark.parametrize("H,H_kv,D", [(64, 8, 128), (40, 8, 128), (56, 8, 64), (80, 16, 64)])
def test_scores_are_as_close_to_64_bits_as_the_vector_kernels(gpu, H, H_kv, D):
    """Root mean square over more than 100000 scores of each: their ratio was 0.98 to 0.99 (1.23 where the sums go from
    product to product); two such means differ by chance by about 1 / sqrt(2 * 100000)."""
    from paper_2411_02886_amd.runtime import to_host
    w = W.make_workload("rms", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[5000], k=64, beta=2.5, planted_per_head=20, seed=9)
    layer, q = make_layer(w)
    kd = layer.k_pool.view(torch.bfloat16).double().cpu()[torch.from_numpy(np.asarray(w.pages_of(0)).astype(np.int64))].view(-1, H_kv, D)[:5000]
    qd = q.view(torch.bfloat16).double().cpu().view(H, D)
    exact = torch.stack([kd[:, h // (H // H_kv)] @ qd[h] for h in range(H)], 1).numpy()
    rms = []
    try:
        for variant in (1, 2):
            gpu.ts_debug_set_score_variant(variant, 0, 0)
            layer.select(q, 1.0, None)
            torch.cuda.synchronize()
            rms.append(float(np.sqrt(np.mean((to_host(layer.scores)[0, :5000].astype(np.float64) - exact) ** 2))))
    finally:
        gpu.ts_debug_set_score_variant(2, 0, 0)
    print("score rms, vector and matrix-core", rms, flush=True)
    assert rms[1] <= 1.02 * rms[0]


@pytest.mark.parametrize("H,H_kv,D,B,max_len,masked,vector", [
    (40, 8, 128, 1, 49152, False, False), (40, 8, 128, 1, 49153, False, True), (56, 8, 64, 2, 49152, False, False), (56, 8, 64, 2, 49153, False, True),
    (48, 8, 128, 3, 49152, True, False), (48, 8, 128, 3, 49153, True, True), (80, 16, 64, 1, 49153, False, True), (64, 8, 128, 1, 49153, False, False),
    (64, 8, 64, 1, 98305, False, False), (64, 8, 128, 2, 65600, True, False), (64, 8, 128, 1, 98305, False, False), (28, 4, 128, 1, 98305, False, False)])
def test_the_score_matrix_on_both_sides_of_its_line(gpu, H, H_kv, D, B, max_len, masked, vector):
    """Five to seven heads over 8 and 16 KV heads take the vector kernel from 96 MiB of K that a call (with a mask: a sequence) may have on.
    Both sides against 64 bits: products are exact, and D - 1 additions of float lose at most 2^-24 of the sum of the absolute
    products each, twice that where they are cut off."""
    from paper_2411_02886_amd.runtime import to_host
    lens = [2049, 33, 700][:B]
    w = W.make_workload("line", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=16, B=B, seq_lens=lens, k=64, beta=2.5, planted_per_head=0, seed=H + B)
    layer, q = make_layer(w, max_seq_len=max_len)
    skip = torch.zeros(B, dtype=torch.uint8, device=q.device) if masked else None
    got = []
    try:
        for mfma in (1, 0):
            gpu.ts_debug_set_codes_path(mfma, 0)
            print("score matrix line", H, H_kv, D, B, max_len, masked, mfma, flush=True)
            layer.select(q, 1.0, skip)
            torch.cuda.synchronize()
            got.append([to_host(layer.scores)[b, :n].copy() for b, n in enumerate(lens)])
    finally:
        gpu.ts_debug_set_codes_path(1, 0)
    assert all(np.array_equal(x, y) for x, y in zip(*got)) == vector
    qf = W.as_f32(w.q, w.dtype).astype(np.float64)
    rows = W.as_f32(w.k_pool.reshape(-1, H_kv, D), w.dtype).astype(np.float64)
    for b in range(B):
        k = np.repeat(rows[w.slots_of(b)], H // H_kv, axis=1)
        exact, size = np.einsum("nhd,hd->nh", k, qf[b, 0]), np.einsum("nhd,hd->nh", np.abs(k), np.abs(qf[b, 0]))
        for x in got:
            assert (np.abs(x[b] - exact) <= 2.0 ** -23 * (D - 1) * size).all()


@pytest.mark.parametrize("H,H_kv,D,P,lens,k", [
    # 513 workgroups of one-tile waves and more: the sequences share the grid (but for the three of 64/16, too few)
    (32, 8, 64, 16, [33000, 32700], 200), (24, 8, 128, 1, [0, 21001, 1, 32, 33, 20000, 129], 300), (28, 4, 64, 16, [40000, 7] + [31] * 14, 64),
    (64, 8, 64, 16, [9000, 12, 17000], 100), (64, 16, 64, 16, [4200, 4097, 4000], 64), (32, 8, 64, 16, list(range(1, 1400, 22)), 40),
    # one sequence too many, and one workgroup too few: each sequence has workgroups of its own
    (32, 8, 64, 16, list(range(0, 1400, 22))[:65] + [1400], 40), (32, 8, 64, 16, [32768, 32768], 64)])
def test_batches_that_share_the_grid(gpu, H, H_kv, D, P, lens, k):
    w = W.make_workload("shared", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=P, B=len(lens), seq_lens=lens, k=k, beta=2.5, planted_per_head=0, seed=k + len(lens))
    for ni, nl in ((0, 0), (4, 61)):
        layer, q = make_layer(w, num_initial=ni, num_local=nl)
        print("shared score grid", H, H_kv, D, P, len(lens), max(lens), ni, nl, flush=True)
        check_compact(w, layer, q, score_scale=1.0, label="shared %dx%d" % (len(lens), max(lens)))


@pytest.mark.parametrize("compact", [False, True], ids=["five-call", "compact"])
@pytest.mark.parametrize("H,H_kv,D,P,lens,max_len", [
    (32, 8, 64, 16, [12000, 0, 9000, 1, 31, 12100, 127, 5000], 12100), (28, 4, 64, 16, [7000] * 9 + [129, 6999], 7000),
    (64, 8, 64, 1, [9000, 40, 8000, 33, 64, 1], 9000), (64, 16, 64, 16, [4200, 65, 4100, 63], 4200),
    # runs of several tiles: the length that the sequences may have decides
    (32, 8, 64, 16, [9000, 257, 0, 700], 150000), (40, 8, 128, 16, [5000, 2049, 31], 70000), (24, 8, 128, 16, [3000, 100], 300000)])
def test_masked_batches_leave_the_statistics_of_each_sequence_alone(gpu, compact, H, H_kv, D, P, lens, max_len):
    """A skip mask or a batch around it changes nothing of a sequence: statistics, index set and count are those of a call of its
    own, bit for bit, and the skipped ones keep theirs."""
    from paper_2411_02886_amd.runtime import to_host
    from paper_2411_02886_amd.runtime import DecodeLayer
    w = W.make_workload("masked", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=P, B=len(lens), seq_lens=lens, k=60, beta=2.5, planted_per_head=0, seed=len(lens) + H)
    layer, q = make_layer(w, max_seq_len=max_len)

    def select(L, q, skip):
        L.idx.fill_(-7); L.count.fill_(-7); L.row_stats.fill_(-3.0)
        (L.select_compact if compact else L.select)(q, 1.0, skip)
        torch.cuda.synchronize()
        return [to_host(x).copy() for x in (L.row_stats, L.idx, L.count)]
    alone = []
    for b in range(len(lens)):
        one = DecodeLayer(dtype=w.dtype, H=H, H_kv=H_kv, D=D, P=P, k=w.k, k_pool=w.k_pool, v_pool=w.v_pool, page_indptr=np.array([0, len(w.pages_of(b))], np.int32),
                          page_indices=w.pages_of(b) if lens[b] else np.zeros(1, np.int32), seq_lens=[lens[b]], max_seq_len=max_len)
        alone.append(select(one, q[b:b + 1].contiguous(), None))
    rng = np.random.default_rng(7)
    masks = [[0] * len(lens)] + [list(rng.integers(0, 2, len(lens))) for _ in range(3)] + [[1] * len(lens)]
    for mask in masks:
        print("masked", H, H_kv, D, mask, flush=True)
        got = select(layer, q, torch.tensor(mask, dtype=torch.uint8, device=q.device))
        for b in range(len(lens)):
            if mask[b]:
                assert (got[0][b] == -3.0).all() and (got[1][b] == -7).all() and got[2][b] == -7, (mask, b)
            else:
                for x, y in zip(got, alone[b]):
                    assert np.array_equal(x[b], y[0], equal_nan=True), (mask, b)


# more work than a tile (a run) per wave of the workgroups that the chip holds: one, two and four wave tiles side by side
_FULL_GRIDS = [(32, 8, 64, [60000, 0, 58123, 33, 41007]), (32, 8, 128, [44000, 45001, 31, 30017]), (28, 4, 128, [52000, 129, 51999, 20000]),
               (64, 8, 64, [30000, 29333, 1, 27041]), (64, 8, 128, [20021, 19000, 21001]), (128, 16, 64, [14000, 13999, 64, 13500]), (96, 32, 64, [14000, 13500, 12777]),
               (40, 8, 64, [23000, 22000, 23456])]


@pytest.mark.parametrize("H,H_kv,D,lens", _FULL_GRIDS)
def test_batches_whose_workgroups_take_several_tiles_per_wave(gpu, H, H_kv, D, lens):
    from rules_util import score_units
    for dense in (False, True):
        assert score_units(len(lens), H, H_kv, D, max(lens), dense, lens, None) > 1
    w = W.make_workload("full", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=16, B=len(lens), seq_lens=lens, k=150, beta=2.5, planted_per_head=0, seed=H + D)
    layer, q = make_layer(w, num_initial=4, num_local=61)
    print("full shared score grid", H, H_kv, D, lens, flush=True)
    check_compact(w, layer, q, score_scale=1.0, label="full %d/%d" % (H, H_kv))


@pytest.mark.parametrize("compact", [False, True], ids=["five-call", "compact"])
@pytest.mark.parametrize("H,H_kv,D,lens,max_len", [c + (max(c[3]),) for c in _FULL_GRIDS] + [(32, 8, 64, [66000, 65000, 45001], 150000)])   # runs of two tiles
def test_masked_batches_of_several_units_per_workgroup(gpu, compact, H, H_kv, D, lens, max_len):
    """The statistics are those of each sequence alone, bit for bit, also where a workgroup forms several units' of them."""
    from rules_util import MASKED, score_shape, score_units
    some = [int(b == 1) for b in range(len(lens))]
    in_pieces = not compact and H_kv >= 8 and 4 < H // H_kv < 8                      # the score matrix of these: a grid of their own
    assert score_shape(len(lens), H, H_kv, D, max_len, not compact, MASKED).shared != in_pieces
    assert in_pieces or score_units(len(lens), H, H_kv, D, max_len, not compact, lens, [0] * len(lens)) > 1
    for mask, (got, alone) in masked_and_alone(H, H_kv, D, 16, lens, max_len, compact, [[0] * len(lens), some]):
        for b in range(len(lens)):
            for x, y in zip(got, alone[b]):
                assert np.array_equal(x[b], np.full_like(x[b], -7 if x.dtype == np.int32 else -3) if mask[b] else y[0], equal_nan=True), (mask, b)


def masked_and_alone(H, H_kv, D, P, lens, max_len, compact, masks):
    from paper_2411_02886_amd.runtime import DecodeLayer, to_host
    w = W.make_workload("masked", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=P, B=len(lens), seq_lens=lens, k=60, beta=2.5, planted_per_head=0, seed=len(lens) + H)
    layer, q = make_layer(w, max_seq_len=max_len)

    def select(L, q, skip):
        L.idx.fill_(-7); L.count.fill_(-7); L.row_stats.fill_(-3.0)
        (L.select_compact if compact else L.select)(q, 1.0, skip)
        torch.cuda.synchronize()
        return [to_host(x).copy() for x in (L.row_stats, L.idx, L.count)]
    alone = []
    for b in range(len(lens)):
        one = DecodeLayer(dtype=w.dtype, H=H, H_kv=H_kv, D=D, P=P, k=w.k, k_pool=layer.k_pool, v_pool=layer.v_pool, page_indptr=np.array([0, len(w.pages_of(b))], np.int32),
                          page_indices=w.pages_of(b) if lens[b] else np.zeros(1, np.int32), seq_lens=[lens[b]], max_seq_len=max_len)
        alone.append(select(one, q[b:b + 1].contiguous(), None))
    for mask in masks:
        print("masked, full grid", H, H_kv, D, mask, flush=True)
        yield mask, (select(layer, q, torch.tensor(mask, dtype=torch.uint8, device=q.device)), alone)


def test_which_batches_share_the_grid():      # no GPU in it, but here stand the lists
    """The launch forms that the lists above stand for."""
    from rules_util import MASKED, WHOLE, score_shape
    for H, H_kv, D, longest, B, shared in [(32, 8, 64, 33000, 2, 1), (24, 8, 128, 21001, 7, 1), (28, 4, 64, 40000, 16, 1), (64, 8, 64, 17000, 3, 1), (64, 16, 64, 4200, 3, 0),
                                           (32, 8, 64, 1387, 64, 1), (32, 8, 64, 1400, 66, 0), (32, 8, 64, 32768, 2, 0)]:
        assert score_shape(B, H, H_kv, D, longest, False, WHOLE).shared == shared, (H, H_kv, D, longest, B)
    for H, H_kv, D, longest, B, dense, shared in [(32, 8, 64, 12100, 8, True, 1), (28, 4, 64, 7000, 11, True, 1), (64, 8, 64, 9000, 6, True, 1), (64, 16, 64, 4200, 4, True, 0),
                                                  (32, 8, 64, 150000, 4, True, 1), (40, 8, 128, 70000, 3, False, 1), (24, 8, 128, 300000, 2, False, 1), (24, 8, 128, 300000, 2, True, 0)]:
        assert score_shape(B, H, H_kv, D, longest, dense, MASKED).shared == shared, (H, H_kv, D, longest, B, dense)
    assert score_shape(3, 40, 8, 128, 70000, True, MASKED) is None                     # the vector kernel


@pytest.mark.parametrize("compact", [False, True], ids=["five-call", "compact"])
@pytest.mark.parametrize("H,H_kv,D,lens,max_len", [(40, 8, 128, [15000, 14001, 65], 30000), (56, 8, 64, [15000, 33, 9001], 99000), (32, 8, 64, [40000, 39001, 1], 40000),
                                                   (128, 16, 64, [3000, 2999], 20000)])
def test_the_cache_test_leaves_the_statistics_of_each_sequence_alone(gpu, compact, H, H_kv, D, lens, max_len):
    """All sequences miss: what the checked call and the vote leave are those of each sequence alone, bit for bit (both sides of the
    line between the kernels)."""
    from paper_2411_02886_amd.runtime import DecodeLayer, to_host
    w = W.make_workload("tested", dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=16, B=len(lens), seq_lens=lens, k=60, beta=2.5, planted_per_head=0, seed=H)
    layer, q = make_layer(w, max_seq_len=max_len)
    layer.first.fill_(1)
    (layer.select_compact if compact else layer.select)(q, 1.0, check_theta=0.9)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        one = DecodeLayer(dtype=w.dtype, H=H, H_kv=H_kv, D=D, P=16, k=w.k, k_pool=layer.k_pool, v_pool=layer.v_pool, page_indptr=np.array([0, len(w.pages_of(b))], np.int32),
                          page_indices=w.pages_of(b), seq_lens=[n], max_seq_len=max_len)
        (one.select_compact if compact else one.select)(q[b:b + 1].contiguous(), 1.0)
        torch.cuda.synchronize()
        for x, y in ((layer.row_stats, one.row_stats), (layer.idx, one.idx), (layer.count, one.count)) + (() if compact else ((layer.scores[:, :n], one.scores[:, :n]),)):
            assert np.array_equal(to_host(x)[b], to_host(y)[0]), b
