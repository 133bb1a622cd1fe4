"""The streaming decode attention on short lists (one run, from one sequence on) and at its lines with splits, against plain
float64 attention: lists of a few keys up to the first split, tiles of 32 keys cut at every kind of remainder, waves without a
tile, forced tokens, an empty sequence beside others."""
import math

import numpy as np
import pytest

import workloads as W
from rules_util import decode_attention

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,H_kv,D,lens,k,ni,nl,streamed", [
    (8, 2, 64, [5], 1, 0, 0, True), (8, 2, 64, [900], 31, 0, 0, True), (12, 2, 128, [900], 32, 0, 0, True),
    (28, 4, 128, [900], 33, 0, 0, True), (32, 8, 128, [900, 40], 96, 4, 29, True), (24, 8, 64, [700, 0, 17], 128, 0, 0, True),
    (8, 2, 64, [900], 256, 0, 0, True), (8, 2, 64, [900], 257, 0, 0, True), (3, 1, 64, [900, 300, 0], 300, 0, 0, True), (28, 4, 128, [900], 320, 0, 0, True),
    (8, 2, 64, [900], 352, 0, 0, False), (64, 8, 128, [900], 257, 0, 0, True),
    (64, 8, 128, [2000] * 3, 1000, 0, 0, True), (28, 4, 128, [2500] * 10, 679, 0, 0, True), (40, 8, 128, [1800] * 6, 1565, 0, 0, True)])
def test_short_lists(H, H_kv, D, lens, k, ni, nl, streamed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2411_02886_amd import binding as ts
    from paper_2411_02886_amd.runtime import DecodeLayer, to_device, to_host
    B, G = len(lens), H // H_kv
    assert decode_attention(B, H, H_kv, D, k + ni + nl)[0] == streamed
    print("short lists", H, H_kv, D, lens, k, ni, nl, flush=True)
    w = W.make_workload("short_lists", dtype=W.BF16, B=B, H=H, H_kv=H_kv, D=D, P=16, seq_lens=lens, k=k, planted_per_head=0, seed=k + H)
    layer = DecodeLayer.from_workload(w, num_initial=ni, num_local=nl)
    rng = np.random.default_rng(k)
    idx, count = np.full((B, k), -1, np.int32), np.zeros(B, np.int32)
    for b, n in enumerate(lens):
        lo = min(ni, n)
        hi = max(lo, n - nl)
        count[b] = min(k, hi - lo)
        idx[b, :count[b]] = np.sort(lo + rng.permutation(hi - lo)[:count[b]])
    layer.idx, layer.count = to_device(idx), to_device(count)
    sm = 1.0 / math.sqrt(D)
    q = np.ascontiguousarray(w.q[0]) if w.q.ndim == 5 else w.q
    layer.out.fill_(3)
    layer.attend(to_device(q), sm)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=True), W.BF16).astype(np.float64).reshape(B, H, D)
    lse = to_host(layer.lse).astype(np.float64).reshape(B, H)
    qf = W.as_f32(q, W.BF16).astype(np.float64).reshape(B, H, D)
    for b, n in enumerate(lens):
        lo = min(ni, n)
        hi = max(lo, n - nl)
        tok = np.concatenate([np.arange(lo), idx[b, :count[b]], np.arange(hi, n)]).astype(int)
        if not len(tok):
            assert not out[b].any() and np.all(np.isneginf(lse[b]))
            continue
        slots = w.slots_of(b)[tok]
        K = W.as_f32(w.k_pool.reshape(-1, H_kv, D)[slots], W.BF16).astype(np.float64)
        V = W.as_f32(w.v_pool.reshape(-1, H_kv, D)[slots], W.BF16).astype(np.float64)
        for h in range(H):
            s = K[:, h // G] @ qf[b, h] * float(np.float32(sm))
            p = np.exp(s - s.max())
            ref = p @ V[:, h // G] / p.sum()
            # float weights and sums; the result's own rounding to bf16
            assert np.abs(out[b, h] - ref).max() <= 2.0 ** -8 * np.abs(ref).max() + 1e-4 * np.abs(V).max(), (b, h)
            assert abs(lse[b, h] - (s.max() + np.log(p.sum()))) <= 1e-5 * max(1.0, np.abs(s).max()), (b, h)
