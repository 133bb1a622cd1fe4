"""The chunk form of the attention against plain float64 attention, where its tiles, splits, row blocks and rescaling
change: key lists of one key up to several tiles per split, row counts around 128, every group size, both head sizes,
scales that are zero, negative or make the logits outgrow the first reference."""
import math

import numpy as np
import pytest

import workloads as W

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CASES = [
    # C, H, H_kv, D, P, cached tokens per sequence, k, n_init, n_local, scale (None = 1/sqrt(D))
    (2, 1, 1, 128, 16, [0], 4, 0, 0, None),
    (16, 8, 1, 128, 16, [1, 0, 63], 64, 0, 0, None),
    (64, 2, 2, 64, 16, [200], 65, 3, 5, None),
    (127, 1, 1, 64, 16, [1000], 128, 0, 0, None),
    (128, 3, 1, 128, 1, [700], 191, 0, 0, 0.0),
    (129, 8, 4, 128, 16, [513, 64], 300, 64, 64, None),
    (43, 24, 8, 128, 16, [900], 517, 0, 0, -0.05),
    (37, 28, 4, 128, 32, [2500, 31, 1200], 1024, 128, 512, None),
    (300, 32, 32, 64, 16, [640], 256, 0, 0, 1.0),
    (512, 16, 2, 128, 16, [4096], 2048, 0, 0, 2.0),
]


@pytest.mark.parametrize("C,H,H_kv,D,P,cached,k,ni,nl,scale", CASES)
def test_chunk_attention(C, H, H_kv, D, P, cached, k, ni, nl, scale):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_02886_amd.runtime import ChunkSelector, to_device, to_host
    print("chunk attention", C, H, H_kv, D, P, cached, k, ni, nl, scale, flush=True)
    w = W.make_workload("chunk", dtype=W.BF16, B=len(cached), C=C, H=H, H_kv=H_kv, D=D, P=P,
                        seq_lens=[n + C for n in cached], k=k, seed=7 * C + D + k)
    layer = ChunkSelector.from_workload(w, num_initial=ni, num_local=nl)
    rng = np.random.default_rng(C)
    idx = np.full((w.B, k), -1, np.int32)
    count = np.zeros(w.B, np.int32)
    for b, n in enumerate(cached):
        lo = min(ni, n)
        hi = max(lo, n - nl)
        count[b] = min(k, hi - lo)
        idx[b, :count[b]] = np.sort(lo + rng.permutation(hi - lo)[:count[b]])
    layer.idx = to_device(idx); layer.count = to_device(count)
    sm = 1.0 / math.sqrt(D) if scale is None else scale
    layer.attend(to_device(w.q), sm)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=True), W.BF16).astype(np.float64)
    lse = to_host(layer.lse).astype(np.float64)
    G = H // H_kv
    q = W.as_f32(w.q, W.BF16).astype(np.float64)
    for b, n in enumerate(cached):
        lo = min(ni, n)
        hi = max(lo, n - nl)
        tok = np.concatenate([np.arange(lo), idx[b, :count[b]], np.arange(hi, n), np.arange(n, n + C)])
        slots = w.slots_of(b)[tok]
        K = W.as_f32(w.k_pool.reshape(-1, H_kv, D)[slots], W.BF16).astype(np.float64)
        V = W.as_f32(w.v_pool.reshape(-1, H_kv, D)[slots], W.BF16).astype(np.float64)
        hidden = np.maximum(np.arange(len(tok)) - (len(tok) - C), -1)[None, :] > np.arange(C)[:, None]
        for h in range(H):
            s = q[b, :, h] @ K[:, h // G].T * float(np.float32(sm))
            s[hidden] = -np.inf
            m = s.max(axis=1, keepdims=True)
            p = np.exp(s - m)
            ref = p @ V[:, h // G] / p.sum(axis=1, keepdims=True)
            ref_lse = m[:, 0] + np.log(p.sum(axis=1))
            # weights rounded to bf16 (2^-9 each, either sign) over values of at most |V|, and the output's own rounding;
            # logits carry float rounding of up to |s| * 2^-22, which acts on a weight as a factor
            tol = (2.0 ** -8 + np.abs(s[~hidden]).max() * 2.0 ** -21) * np.abs(V[:, h // G]).max()
            assert np.abs(out[b, :, h] - ref).max() <= tol, (b, h)
            assert np.abs(lse[b, :, h] - ref_lse).max() <= 2.0 ** -8 + np.abs(s[~hidden]).max() * 2.0 ** -20, (b, h)


@pytest.mark.parametrize("k", [60, 700], ids=["one-split", "splits"])
def test_stale_and_corrupt_selection_state(k):
    """Token ids outside the sequence are clamped into it, counts into [0, k]; a sequence shorter than the chunk holds none."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_02886_amd.runtime import ChunkSelector, to_device, to_host
    C, H, H_kv, D = 20, 8, 2, 128
    cached = [k + 11, k, 5, -20]                            # the last one is empty
    w = W.make_workload("stale_chunk", dtype=W.BF16, B=4, C=C, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[n + C for n in cached], k=k, seed=8)
    layer = ChunkSelector.from_workload(w)
    rng = np.random.default_rng(k)
    idx = rng.integers(0, k, size=(4, k)).astype(np.int32)
    count = np.array([k, k + 500, -4, k], np.int32)
    idx[0, 3] = -12; idx[0, 5] = 10 ** 9; idx[1, 7] = -2 ** 31; idx[1, k - 1] = 2 ** 31 - 1
    layer.idx = to_device(idx); layer.count = to_device(count)
    print("stale chunk selection", k, flush=True)
    sm = 1.0 / math.sqrt(D)
    layer.out.fill_(3)
    layer.attend(to_device(w.q), sm)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=True), W.BF16).astype(np.float64)
    assert not out[3].any()
    for b, n in enumerate(cached[:3]):
        att = np.clip(idx[b, :min(max(int(count[b]), 0), k)], 0, n + C - 1)
        slots = w.slots_of(b)
        for c in (0, C - 1):
            tok = slots[np.concatenate([att, np.arange(n, n + c + 1)])]
            K = W.as_f32(w.k_pool.reshape(-1, H_kv, D)[tok], W.BF16).astype(np.float64)
            V = W.as_f32(w.v_pool.reshape(-1, H_kv, D)[tok], W.BF16).astype(np.float64)
            for h in range(H):
                s = K[:, h // 4] @ W.as_f32(w.q[b, c, h], W.BF16).astype(np.float64) * sm
                p = np.exp(s - s.max())
                assert np.abs(out[b, c, h] - p @ V[:, h // 4] / p.sum()).max() <= 2.0 ** -7 * np.abs(V).max(), (b, c, h)
