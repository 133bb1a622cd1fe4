"""The chunk attention (head size 128: four waves of 64 rows; 64: eight of 32; two key groups) where its pipeline changes shape: key lists that
end at, before and after a tile of either key group, and logits that jump up in a chosen tile -- a raised reference in an
even or odd tile, in its first or second half, and one so large that the loop without masks ends there."""
import math

import numpy as np
import pytest

import workloads as W
from rules_util import rules

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _attend(C, H, H_kv, D, cached, n_init, spikes, sign=1.0):
    """One sequence whose `cached` tokens are all selected (or forced); spikes: {list position: logit of every query with that key};
    sign: of the softmax scale."""
    from paper_2411_02886_amd.runtime import ChunkSelector, to_device, to_host
    k = max(1, cached - n_init)
    w = W.make_workload("wide", dtype=W.BF16, B=1, C=C, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[cached + C], k=k, seed=3 * cached + C)
    sm = sign / math.sqrt(D)
    slots = w.slots_of(0)
    if spikes:
        # query = a common direction plus a little noise across it: the spikes' logits are the same for all queries and exact
        q = W.as_f32(w.q, W.BF16)
        q[..., :8] = 0.0
        q[..., 0] = 8.0
        w.q[:] = W.f32_to_bf16_bits(q)
        rows = W.as_f32(w.k_pool.reshape(-1, H_kv, D), W.BF16)
        rows[:, :, :8] = 0.0
        for pos, logit in spikes.items():
            rows[slots[pos]] = 0.0
            rows[slots[pos], :, 0] = logit / sm / 8.0
        w.k_pool[:] = W.f32_to_bf16_bits(rows).reshape(w.k_pool.shape)
    layer = ChunkSelector.from_workload(w, num_initial=n_init)
    idx = np.arange(n_init, n_init + k, dtype=np.int32)[None]
    layer.idx = to_device(idx); layer.count = to_device(np.array([cached - n_init], np.int32))
    layer.attend(to_device(w.q), sm)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=True), W.BF16).astype(np.float64)[0]
    lse = to_host(layer.lse).astype(np.float64)[0]
    q = W.as_f32(w.q, W.BF16).astype(np.float64)[0]
    K = W.as_f32(w.k_pool.reshape(-1, H_kv, D)[slots[:cached + C]], W.BF16).astype(np.float64)
    V = W.as_f32(w.v_pool.reshape(-1, H_kv, D)[slots[:cached + C]], W.BF16).astype(np.float64)
    hidden = np.maximum(np.arange(cached + C) - cached, -1)[None, :] > np.arange(C)[:, None]
    for h in range(H):
        s = q[:, h] @ K[:, h * H_kv // H].T * float(np.float32(sm))
        s[hidden] = -np.inf
        m = s.max(axis=1, keepdims=True)
        p = np.exp(s - m)
        ref = p @ V[:, h * H_kv // H] / p.sum(axis=1, keepdims=True)
        # logits near the largest decide; theirs is the rounding that acts on the weights (of up to |s| * 2^-22), besides the
        # weights' own to bf16 (2^-9) and the output's
        near = np.abs(m).max() * (2.0 ** -21 if np.abs(m).max() < 2.0 ** 12 else 0.0)
        tol = (2.0 ** -8 + near) * np.abs(V[:, h * H_kv // H]).max()
        assert np.abs(out[:, h] - ref).max() <= tol, h
        ref_lse = m[:, 0] + np.log(p.sum(axis=1))
        assert np.abs(lse[:, h] - ref_lse).max() <= 2.0 ** -8 + np.abs(m).max() * 2.0 ** -20, h


@pytest.mark.parametrize("cached", [1, 31, 62, 63, 64, 94, 126, 127, 128, 190, 191, 254, 255, 319, 383, 447, 1151])
@pytest.mark.parametrize("C,H,H_kv,D", [(2, 3, 1, 128), (33, 8, 2, 128), (33, 8, 2, 64)])
def test_key_lists_around_the_tiles(cached, C, H, H_kv, D):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    print("wide chunk attention", cached, C, H, H_kv, D, flush=True)
    _attend(C, H, H_kv, D, cached, 0, {})


# Logits of the spikes against ordinary ones of a few units.  160 queries of two heads are three row blocks, whose lists of 700 +
# 64, 128 or 160 keys are cut into three splits of four, five and five tiles; a key group has every other one of them.  The last
# spike's is the largest by far, so that one key decides where the logits are so large that their float rounding is not small.
SPIKES = [{70: 30.0}, {200: 40.0}, {64 * 4 + 3: 60.0, 64 * 5 + 40: 90.0}, {0: 25.0, 64 * 7 + 33: 80.0}, {64 * 3 + 35: 2.0 ** 22},
          {64 * 2: 2.0 ** 21, 64 * 6 + 1: 2.0 ** 23}, {64 * 10 + 63: 50.0}]


@pytest.mark.parametrize("spikes", SPIKES, ids=range(len(SPIKES)))
@pytest.mark.parametrize("n_init,D", [(0, 128), (37, 128), (0, 64)])
def test_references_raised_in_either_group_and_half(spikes, n_init, D):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert rules().rule_chunk_splits(160, 2, 1, D, 700 - n_init, n_init) == 3
    print("wide chunk attention, spikes", spikes, n_init, D, flush=True)
    _attend(160, 2, 1, D, 700, n_init, spikes)


# The line from which logits are rounded (2^20, base two) is passed in the second half of a tile in the loop without masks, and
# the next block, the first half of the key group's next tile, whose scores are there by then, holds a large one too: a smaller,
# an equal, a larger one.  A key group's first tile is left out (its two halves are looked at together).  700 keys, as above: the even
# group of the first split has tiles 0, 2, 4, of the second 5, 7, 9; 3100 keys, eight splits of seven tiles: the odd one 1, 3, 5.
LARGE = [(700, {64 * 2 + 37: 2.0 ** 22, 64 * 4 + 1: 2.0 ** 21}), (700, {64 * 2 + 37: 2.0 ** 22, 64 * 4 + 1: 2.0 ** 22}),
         (700, {64 * 2 + 63: 2.0 ** 21, 64 * 4 + 31: 2.0 ** 22}), (700, {64 * 7 + 32: 2.0 ** 23, 64 * 9: 2.0 ** 22}),
         (3100, {64 * 3 + 35: 2.0 ** 21, 64 * 5 + 3: 2.0 ** 20 * 1.5}), (3100, {64 * 3 + 32: 2.0 ** 22, 64 * 5 + 31: 2.0 ** 22})]


@pytest.mark.parametrize("cached,spikes", LARGE, ids=range(len(LARGE)))
@pytest.mark.parametrize("D,sign", [(128, 1.0), (128, -1.0), (64, 1.0)])
def test_logits_are_rounded_from_the_block_on_that_passes_the_line(cached, spikes, D, sign):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert rules().rule_chunk_splits(160, 2, 1, D, cached, 0) == (3 if cached == 700 else 8)
    print("wide chunk attention, large logits", cached, spikes, D, sign, flush=True)
    _attend(160, 2, 1, D, cached, 0, spikes, sign=sign)
