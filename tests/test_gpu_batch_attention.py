"""Both batch forms of the decode attention against plain float64 attention.  Streaming (bf16): runs of one key, of less
and more than a tile, of several splits; every group size; scales that are zero, negative or make the logits outgrow the
first reference; empty sequences beside full ones.  Several 64-token chunks per workgroup (fp32, and bf16 with one or two
heads per KV head): a last workgroup of one to four chunks, empty splits, forced tokens, up to eight heads."""
import math

import numpy as np
import pytest

import workloads as W
from rules_util import decode_attention

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # B, H, H_kv, D, P, longest sequence, k, n_init, n_local, scale (None = 1/sqrt(D))
    (256, 8, 8, 64, 16, 200, 129, 0, 0, None),
    (300, 14, 2, 128, 16, 400, 257, 3, 5, None),
    (96, 32, 16, 128, 1, 300, 129, 0, 0, 0.0),
    (40, 24, 8, 64, 16, 700, 500, 4, 61, -0.3),
    (12, 32, 8, 128, 16, 3000, 2048, 128, 512, None),
    (10, 40, 8, 128, 32, 2000, 1777, 0, 0, 2.0),
    (33, 12, 2, 128, 16, 2300, 2100, 0, 0, 1.0),
    (3, 32, 4, 128, 16, 12000, 11000, 0, 0, None),
    (9, 64, 8, 64, 16, 1900, 1800, 0, 0, 0.5),
]


CHUNKED = [
    # dtype, then as above: 8192 chunk workgroups and more, counted over lists of k entries
    (W.F32, 33, 16, 8, 128, 16, 700, 2000, 0, 0, None),
    (W.F32, 35, 16, 8, 128, 16, 600, 1900, 10, 50, None),
    (W.F32, 70, 20, 4, 64, 4, 450, 1870, 3, 61, 1.0),
    (W.F32, 66, 32, 4, 128, 16, 330, 2000, 0, 0, -0.3),
    (W.F32, 9, 16, 16, 64, 1, 1500, 4096, 4, 0, None),
    (W.BF16, 33, 16, 8, 64, 16, 700, 2000, 10, 50, None),
    (W.BF16, 18, 16, 16, 128, 16, 900, 2048, 0, 0, None),
]


@pytest.mark.parametrize("B,H,H_kv,D,P,longest,k,ni,nl,scale", CASES)
def test_batch_attention(B, H, H_kv, D, P, longest, k, ni, nl, scale):
    assert decode_attention(B, H, H_kv, D, k + ni + nl)[0], "not streamed"
    check_batch(W.BF16, B, H, H_kv, D, P, longest, k, ni, nl, scale)


@pytest.mark.parametrize("dtype,B,H,H_kv,D,P,longest,k,ni,nl,scale", CHUNKED)
def test_batch_attention_in_chunks(dtype, B, H, H_kv, D, P, longest, k, ni, nl, scale):
    assert (k + ni + nl + 63) // 64 * H_kv * B >= 8192
    assert dtype == W.F32 or not decode_attention(B, H, H_kv, D, k + ni + nl)[0], "streamed"
    check_batch(dtype, B, H, H_kv, D, P, longest, k, ni, nl, scale)


def check_batch(dtype, B, H, H_kv, D, P, longest, k, ni, nl, scale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_02886_amd.runtime import DecodeLayer, to_device, to_host
    print("batch attention", dtype, B, H, H_kv, D, P, longest, k, ni, nl, scale, flush=True)
    rng = np.random.default_rng(B + k)
    lens = rng.integers(1, longest + 1, size=B)
    lens[0], lens[-1] = longest, (0 if B > 3 else 1)
    w = W.make_workload("batch", dtype=dtype, B=B, H=H, H_kv=H_kv, D=D, P=P, seq_lens=lens, k=k, seed=3 * B + D + k)
    layer = DecodeLayer.from_workload(w, num_initial=ni, num_local=nl)
    idx = np.full((B, k), -1, np.int32)
    count = np.zeros(B, np.int32)
    for b, n in enumerate(int(x) for x in lens):
        lo = min(ni, n)
        hi = max(lo, n - nl)
        count[b] = min(k, hi - lo)
        idx[b, :count[b]] = np.sort(lo + rng.permutation(hi - lo)[:count[b]])
    layer.idx = to_device(idx); layer.count = to_device(count)
    sm = 1.0 / math.sqrt(D) if scale is None else scale
    layer.attend(to_device(w.q), sm)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=dtype == W.BF16), dtype).astype(np.float64)
    lse = to_host(layer.lse).astype(np.float64)
    G = H // H_kv
    q = W.as_f32(w.q, dtype).astype(np.float64)
    for b in sorted(set([0, B - 1, B - 2] + list(rng.integers(0, B, size=5)))):
        n = int(lens[b])
        if n == 0:
            assert not out[b].any() and np.all(np.isneginf(lse[b])), b
            continue
        lo = min(ni, n)
        tok = np.concatenate([np.arange(lo), idx[b, :count[b]], np.arange(max(lo, n - nl), n)])
        slots = w.slots_of(b)[tok]
        K = W.as_f32(w.k_pool.reshape(-1, H_kv, D)[slots], dtype).astype(np.float64)
        V = W.as_f32(w.v_pool.reshape(-1, H_kv, D)[slots], dtype).astype(np.float64)
        for h in range(H):
            s = K[:, h // G] @ q[b, 0, h] * float(np.float32(sm))
            p = np.exp(s - s.max())
            ref = p @ V[:, h // G] / p.sum()
            # the weights are float (the output's rounding to bf16 is 2^-9 of it); logits carry float rounding of up to
            # |s| * 2^-22, which acts on a weight as a factor
            err = np.abs(s).max() * 2.0 ** -21 + 2.0 ** -20
            if dtype == W.F32:
                err += 2.0 ** -19            # the float sums over V: chains of up to 32 additions, 2^-24 each
            own = 2.0 ** (-8 if dtype == W.BF16 else -22)
            assert np.all(np.abs(out[b, 0, h] - ref) <= own * np.abs(ref) + err * np.abs(V[:, h // G]).max()), (b, h)
            assert abs(lse[b, 0, h] - (s.max() + math.log(p.sum()))) <= err + np.abs(s).max() * 2.0 ** -22, (b, h)


# ---- what the smaller batches of the other files do not reach with these forms: stale selections, non-finite inputs, capture,
# pools beyond 4 GiB.  dtype, B, H, H_kv, D, longest, k; streamed without and with splits, and in runs of chunks
FORMS = {"streamed": (W.BF16, 26, 40, 8, 64, 340, 300), "streamed-splits": (W.BF16, 9, 32, 8, 128, 2100, 2000),
         "chunk-runs": (W.F32, 33, 16, 8, 64, 330, 2000)}


def make_batch(form, lens=None):
    from paper_2411_02886_amd.runtime import DecodeLayer, to_device
    dtype, B, H, H_kv, D, longest, k = FORMS[form]
    rng = np.random.default_rng(B)
    if lens is None:
        lens = rng.integers(1, longest + 1, size=B)
        lens[0] = longest
    streamed, splits = decode_attention(B, H, H_kv, D, k)
    assert form == "chunk-runs" or (streamed and (splits > 1) == (form == "streamed-splits"))
    w = W.make_workload("form", dtype=dtype, B=B, H=H, H_kv=H_kv, D=D, P=16, seq_lens=lens, k=k, seed=31 + B)
    layer = DecodeLayer.from_workload(w)
    idx = np.full((B, k), -1, np.int32)
    count = np.minimum(np.asarray(lens), k).astype(np.int32)
    for b, n in enumerate(int(x) for x in lens):
        idx[b, :count[b]] = np.sort(rng.permutation(n)[:count[b]])
    layer.idx, layer.count = to_device(idx), to_device(count)
    return w, layer, to_device(w.q), idx, count


def check_outputs(w, layer, idx, count, sequences):
    """Against float64, with the same reading of the selection as the kernels': ids clamped into the sequence."""
    from paper_2411_02886_amd.runtime import to_host
    out = W.as_f32(to_host(layer.out, bits16=w.dtype == W.BF16), w.dtype).astype(np.float64)
    sm, G = 1.0 / math.sqrt(w.D), w.H // w.H_kv
    for b in sequences:
        n = int(w.seq_lens[b])
        if n == 0:
            assert not out[b].any(), b
            continue
        slots = w.slots_of(b)[np.clip(idx[b, :min(max(int(count[b]), 0), w.k)], 0, n - 1)]
        K = W.as_f32(w.k_pool.reshape(-1, w.H_kv, w.D)[slots], w.dtype).astype(np.float64)
        V = W.as_f32(w.v_pool.reshape(-1, w.H_kv, w.D)[slots], w.dtype).astype(np.float64)
        for h in range(w.H):
            s = K[:, h // G] @ W.as_f32(w.q[b, 0, h], w.dtype).astype(np.float64) * sm
            p = np.exp(s - s.max())
            assert np.abs(out[b, 0, h] - p @ V[:, h // G] / p.sum()).max() <= 2.0 ** -8 * np.abs(V).max(), (b, h)


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02886_amd as ts
    ts.load()
    return ts


@pytest.mark.parametrize("form", list(FORMS))
def test_stale_and_corrupt_selection_state(gpu, form):
    """Token ids outside the sequence, counts above k and below zero, a count on an empty sequence (which owns no page)."""
    from paper_2411_02886_amd.runtime import to_device
    _, B, _, _, _, longest, k = FORMS[form]
    lens = np.full(B, min(longest, k) - 20, int)
    lens[2] = lens[B - 1] = 0
    w, layer, q, idx, count = make_batch(form, lens)
    idx[0, 3] = -12; idx[0, 5] = 10 ** 9; idx[1, 0] = lens[1]; idx[1, 200] = -2 ** 31
    count[1] = k + 1000; idx[1, lens[1]:] = 2 ** 31 - 1
    count[2] = 17; idx[2, :17] = 5
    count[B - 1] = k
    count[4] = -3; count[5] = 1
    layer.idx.copy_(to_device(idx)); layer.count.copy_(to_device(count))
    print("stale selection", form, flush=True)
    layer.out.fill_(3)
    layer.attend(q, 1.0 / math.sqrt(w.D))
    torch.cuda.synchronize()
    w.seq_lens[4] = 0                                     # a negative count selects nothing: rows are zero as well
    check_outputs(w, layer, idx, count, range(6))
    check_outputs(w, layer, idx, count, [B - 1])


@pytest.mark.parametrize("form", list(FORMS))
def test_nonfinite_inputs(gpu, form):
    """Results are unspecified, but the calls complete, other sequences keep theirs, and the layer is healthy afterwards."""
    from test_gpu_nonfinite_inputs import poison
    w, layer, q, idx, count = make_batch(form)
    B = w.B
    rng = np.random.default_rng(6)
    saved = layer.k_pool.clone(), layer.v_pool.clone()
    row = w.H_kv * w.D
    for what in ("nan", "inf", "-inf"):
        print("nonfinite batch", form, what, flush=True)
        for pool in (layer.k_pool, layer.v_pool):         # rows of the first two sequences only
            slots = np.concatenate([rng.choice(w.slots_of(b), 5) for b in (0, 1)])
            poison(pool, w.dtype, torch.from_numpy(slots * row + rng.integers(0, row, slots.size)).to(q.device), what)
        layer.attend(q, 1.0 / math.sqrt(w.D))
        torch.cuda.synchronize()
        check_outputs(w, layer, idx, count, [2, B // 2, B - 1])
    layer.k_pool.copy_(saved[0]); layer.v_pool.copy_(saved[1])
    layer.attend(q, 1.0 / math.sqrt(w.D))
    torch.cuda.synchronize()
    check_outputs(w, layer, idx, count, [0, 1, B - 1])


@pytest.mark.parametrize("form", list(FORMS))
def test_capture(gpu, form):
    from test_gpu_graph_capture import capture_and_replay
    w, layer, q, idx, count = make_batch(form)
    print("captured batch", form, flush=True)
    capture_and_replay(lambda: layer.attend(q, 1.0 / math.sqrt(w.D)), [layer.out, layer.lse],
                       lambda: (layer.out.zero_(), layer.lse.fill_(3.0)))
    check_outputs(w, layer, idx, count, [0, 1, w.B - 1])


@pytest.mark.parametrize("form", list(FORMS))
def test_pools_beyond_4_gib(gpu, form):
    from test_gpu_large_pool import spread_over_large_pools
    w, layer, q, idx, count = make_batch(form)
    wl = spread_over_large_pools(w, seed=2)
    from paper_2411_02886_amd.runtime import DecodeLayer
    big = DecodeLayer.from_workload(wl)
    big.idx, big.count = layer.idx, layer.count
    print("large pool batch", form, flush=True)
    big.attend(q, 1.0 / math.sqrt(w.D))
    torch.cuda.synchronize()
    check_outputs(w, big, idx, count, [0, 1, w.B - 1])
    del big, wl
    torch.cuda.empty_cache()
