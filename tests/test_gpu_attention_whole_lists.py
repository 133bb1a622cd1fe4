"""Decode attention of lists of up to 256 entries by one workgroup (fp32, and bf16 of one and two heads per KV head) against plain
float64 attention: every kind of remainder, the first list that is split, forced tokens, empty sequences, an infinite value."""
import numpy as np
import pytest

import workloads as W
from test_gpu_batch_attention import check_batch

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,H,H_kv,D", [(W.F32, 8, 2, 64), (W.F32, 7, 1, 64), (W.F32, 64, 8, 64), (W.F32, 3, 1, 128), (W.F32, 8, 8, 128),
                                            (W.BF16, 2, 2, 64), (W.BF16, 8, 4, 128), (W.BF16, 4, 2, 64)])
@pytest.mark.parametrize("B,longest,k,ni,nl", [(2, 40, 1, 0, 0), (3, 300, 15, 0, 0), (5, 300, 16, 4, 45), (4, 400, 128, 0, 0), (9, 500, 255, 0, 0),
                                               (4, 500, 150, 45, 61), (2, 500, 257, 0, 0)])
def test_whole_lists(dtype, H, H_kv, D, B, longest, k, ni, nl):
    check_batch(dtype, B, H, H_kv, D, 16, longest, k, ni, nl, None)


@pytest.mark.parametrize("dtype,H,H_kv,D,B,longest,k,ni,nl", [(W.F32, 8, 2, 64, 6, 240, 60, 100, 20), (W.F32, 8, 2, 64, 9, 600, 200, 150, 45),
                                                              (W.F32, 7, 1, 128, 70, 700, 300, 200, 61), (W.BF16, 28, 4, 128, 3, 400, 260, 390, 0)])
def test_fewer_tokens_than_forced_ones(dtype, H, H_kv, D, B, longest, k, ni, nl):
    """The list is loaded as if all forced tokens were there; sequences shorter than that (whole list, splits, runs of chunks)."""
    check_batch(dtype, B, H, H_kv, D, 16, longest, k, ni, nl, None)


@pytest.mark.parametrize("dtype,H,H_kv,D", [(W.F32, 8, 2, 64), (W.BF16, 4, 2, 128)])
def test_an_infinite_value_in_a_short_list(dtype, H, H_kv, D):
    """The list's first row stands in for the padding: an infinity there comes out infinite, and only in its own place."""
    from paper_2411_02886_amd.runtime import DecodeLayer, to_device, to_host
    w = W.make_workload("inf", dtype=dtype, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[60], k=9, seed=5)
    layer = DecodeLayer.from_workload(w)
    layer.idx = to_device(np.arange(10, 19, dtype=np.int32)[None]); layer.count = to_device(np.array([9], np.int32))
    v = layer.v_pool.view(torch.bfloat16 if dtype == W.BF16 else torch.float32).view(-1, H_kv, D)
    v[int(w.slots_of(0)[10]), 0, 3] = float("inf")
    layer.attend(to_device(w.q), 0.1)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=dtype == W.BF16), dtype).reshape(H, D)
    G = H // H_kv
    assert np.all(np.isposinf(out[:G, 3]))
    out[:G, 3] = 0
    assert np.all(np.isfinite(out))
