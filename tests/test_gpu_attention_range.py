"""The attention kernels at the ends of the number range, against plain float64: logits of any finite size, values up to
what a sum of them can hold, and the log-sum-exp of the streaming form against that of the form it stands in for."""
import math

import numpy as np
import pytest

import workloads as W
from rules_util import decode_attention

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# form: B, C, H, H_kv, D, tokens before the chunk (all of them selected)
FORMS = {
    "chunks": (1, 1, 8, 2, 64, 400),
    "streamed-one-run": (1, 1, 8, 2, 64, 300),
    "streamed": (26, 1, 40, 8, 64, 300),
    "streamed-splits": (2, 1, 64, 8, 128, 4096),
    "chunk-form": (1, 24, 8, 2, 128, 250),
    "chunk-form-splits": (1, 48, 8, 2, 64, 1000),
}
STREAMED = {"chunks": (False, 7), "streamed-one-run": (True, 1), "streamed": (True, 1), "streamed-splits": (True, 16)}


@pytest.fixture(scope="module")
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2411_02886_amd as ts
    ts.load()
    return ts


def attend(form, K, q, V, sm):
    """Attention of every head over all tokens, with the same key rows K [n][D], query row q [D] and value rows V [n][D]
    everywhere.  Returns (out, lse) of the last sequence as float64 [C][H][D], [C][H] and the references [C][D], [C]."""
    from paper_2411_02886_amd.runtime import ChunkSelector, DecodeLayer, to_device, to_host
    B, C, H, H_kv, D, cached = FORMS[form]
    n = cached + (C if C > 1 else 0)
    if C == 1:
        assert decode_attention(B, H, H_kv, D, cached) == STREAMED[form]
    w = W.make_workload("range", dtype=W.BF16, B=B, C=C, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[n] * B, k=cached, seed=5)
    bits = lambda x: W.store(np.asarray(x, np.float32), W.BF16)
    for x in (K, q, V):
        fin = np.isfinite(x)
        assert np.array_equal(W.as_f32(bits(x), W.BF16)[fin], np.asarray(x, np.float32)[fin])     # bf16 numbers as they are
    for b in range(B):
        w.k_pool.reshape(-1, H_kv, D)[w.slots_of(b)] = bits(K)[:, None]
        w.v_pool.reshape(-1, H_kv, D)[w.slots_of(b)] = bits(V)[:, None]
    w.q[:] = bits(q)
    layer = (DecodeLayer if C == 1 else ChunkSelector).from_workload(w)
    layer.idx = to_device(np.tile(np.arange(cached, dtype=np.int32), (B, 1)))
    layer.count = to_device(np.full(B, cached, np.int32))
    layer.attend(to_device(w.q), sm)
    torch.cuda.synchronize()
    out = W.as_f32(to_host(layer.out, bits16=True), W.BF16).astype(np.float64)[-1]
    lse = to_host(layer.lse).astype(np.float64)[-1]
    s = (K.astype(np.float64) @ q.astype(np.float64)) * float(np.float32(sm))
    ref, ref_lse = [], []
    for c in range(C):
        m = n if C == 1 else cached + c + 1
        p = np.exp(s[:m] - s[:m].max())
        with np.errstate(invalid="ignore"):
            ref.append((p[:, None] * V[:m].astype(np.float64)).sum(axis=0) / p.sum())
        ref_lse.append(s[:m].max() + math.log(p.sum()))
    return out, lse, np.array(ref), np.array(ref_lse)


def rows(form):
    _, C, _, _, D, cached = FORMS[form]
    return cached + (C if C > 1 else 0), D


def bf16_values(rng, shape):
    return W.as_f32(W.store(rng.standard_normal(shape).astype(np.float32), W.BF16), W.BF16)


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("exponent", [20, 28, 36, 105, 124])
@pytest.mark.parametrize("sign", [1, -1])
def test_large_logits(gpu, form, exponent, sign):
    """Logits of about 2^exponent, all of one sign, in 61 classes of equal ones a 64th apart: far apart beside their own
    rounding, so that the weights are those of the largest class alone."""
    n, D = rows(form)
    print("large logits", form, exponent, sign, flush=True)
    K, q = np.zeros((n, D), np.float32), np.zeros(D, np.float32)
    q[0] = 2.0 ** (exponent // 2)
    K[:, 0] = sign * 2.0 ** (exponent - exponent // 2) * (1 + (np.arange(n) * 7 % 61) / 64)
    V = bf16_values(np.random.default_rng(exponent), (n, D))
    out, lse, ref, ref_lse = attend(form, K, q, V, 0.3)
    # weights of 0 and 1 (exact in bf16 too), sums of up to 100 values, the result's rounding to bf16
    assert np.abs(out - ref[:, None]).max() <= 2.0 ** -8 * np.abs(ref).max() + 2.0 ** -16
    assert np.abs(lse - ref_lse[:, None]).max() <= 2.0 ** -22 * np.abs(ref_lse).max()


# Exponent of V's elements: weights of at most 1 over 300 to 4096 keys fit a float.  The chunk forms raise their reference at a weight of
# 2, so that weights below that over 274 keys (2^(1 + 8.1 + 118)), and over the 1048 keys of the other (2^(1 + 10.1 + 116)), fit too.
LARGE_VALUES = {"chunks": 118, "streamed-one-run": 118, "streamed": 118, "streamed-splits": 115, "chunk-form": 118, "chunk-form-splits": 116}


@pytest.mark.parametrize("form", list(FORMS))
@pytest.mark.parametrize("rise", [13.25, 10.5, 5.75])
def test_large_values_under_rising_logits(gpu, form, rise):
    """Every other stretch of 128 keys has logits 19, 15 or 8 octaves above the rest: less than a float holds, so that a kernel may
    leave its reference where it was, but then its weights must not outgrow the room above the values."""
    n, D = rows(form)
    print("large values", form, rise, flush=True)
    K, q = np.zeros((n, D), np.float32), np.zeros(D, np.float32)
    q[0] = 1.0
    K[:, 0] = np.where(np.arange(n) // 128 % 2 == 1, rise, 0.0)
    V = np.ldexp(1 + np.abs(bf16_values(np.random.default_rng(3), (n, D))) % 1.0, LARGE_VALUES[form] - 1)
    V = W.as_f32(W.store(V.astype(np.float32), W.BF16), W.BF16)
    out, lse, ref, ref_lse = attend(form, K, q, V, 1.0)
    assert np.isfinite(out).all()
    # all of V's elements have one sign: the weights' rounding to bf16 (chunk form) and the result's own
    assert np.abs(out / ref[:, None] - 1).max() <= 2.0 ** -7
    assert np.abs(lse - ref_lse[:, None]).max() <= 2.0 ** -8


@pytest.mark.parametrize("form", list(FORMS))
def test_infinite_values(gpu, form):
    """A value row with infinite elements under a weight that is not zero: those elements of the output are infinite, the
    others what they are without it."""
    n, D = rows(form)
    print("infinite values", form, flush=True)
    rng = np.random.default_rng(4)
    K, q, V = bf16_values(rng, (n, D)), bf16_values(rng, D), bf16_values(rng, (n, D))
    for t, d, x in ((37, 3, np.inf), (70, 5, -np.inf), (71, D - 1, np.inf), (222, 3, np.inf)):
        V[t, d] = x
    out, lse, ref, ref_lse = attend(form, K, q, V, 1.0 / math.sqrt(D))
    assert np.array_equal(np.isinf(out[:, 0]), np.isinf(ref)) and np.array_equal(np.isnan(out), np.zeros(out.shape, bool))
    inf = np.isinf(ref)
    for h in range(out.shape[1]):
        assert np.array_equal(out[:, h][inf], ref[inf])
        # weights rounded to bf16 in the chunk form, the result's own rounding
        assert np.abs(out[:, h][~inf] - ref[~inf]).max() <= 2.0 ** -7 * np.abs(V[np.isfinite(V)]).max()


@pytest.mark.parametrize("H,H_kv,D,k,scale", [(32, 8, 128, 2048, 1.0), (28, 4, 128, 1500, 4.0), (24, 8, 64, 1000, 4.0), (64, 8, 64, 600, 1.0)])
def test_log_sum_exp_of_the_streaming_form_is_as_close_as_that_of_the_chunks(gpu, H, H_kv, D, k, scale):
    """The same sequences attended as a batch (streamed) and one by one (64-token chunks): the root mean square of the
    log-sum-exp's distance from float64 over all heads may not be larger, but for what 10 % of chance in it leaves."""
    from paper_2411_02886_amd.runtime import DecodeLayer, to_device, to_host
    B = max(1, 2600 // ((k + 63) // 64 * H_kv)) + 1
    assert decode_attention(B, H, H_kv, D, k)[0] and not decode_attention(1, H, H_kv, D, k)[0]
    print("lse", H, H_kv, D, k, scale, B, flush=True)
    w = W.make_workload("lse", dtype=W.BF16, B=B, H=H, H_kv=H_kv, D=D, P=16, seq_lens=[k] * B, k=k, seed=9)
    sm = float(np.float32(scale / math.sqrt(D)))
    layer = DecodeLayer.from_workload(w)
    idx = to_device(np.tile(np.arange(k, dtype=np.int32), (B, 1)))
    layer.idx, layer.count = idx, to_device(np.full(B, k, np.int32))
    q = to_device(w.q)
    layer.attend(q, sm)
    torch.cuda.synchronize()
    got = {"streamed": to_host(layer.lse).astype(np.float64)[:, 0], "chunks": np.empty((B, H))}
    want = np.empty((B, H))
    for b in range(B):
        one = DecodeLayer(dtype=W.BF16, H=H, H_kv=H_kv, D=D, P=16, k=k, k_pool=layer.k_pool, v_pool=layer.v_pool,
                          page_indptr=[0, len(w.pages_of(b))], page_indices=w.pages_of(b), seq_lens=[k])
        one.idx, one.count = idx[:1].contiguous(), to_device(np.array([k], np.int32))
        one.attend(q[b:b + 1].contiguous(), sm)
        got["chunks"][b] = to_host(one.lse).astype(np.float64)[0, 0]
        K = W.as_f32(w.k_pool.reshape(-1, H_kv, D)[w.slots_of(b)], W.BF16).astype(np.float64)
        qb = W.as_f32(w.q[b, 0], W.BF16).astype(np.float64)
        for h in range(H):
            s = K[:, h // (H // H_kv)] @ qb[h] * sm
            want[b, h] = s.max() + math.log(np.exp(s - s.max()).sum())
    rms = {f: float(np.sqrt(((got[f] - want) ** 2).mean())) for f in got}
    print("rms error of the log-sum-exp: streamed %.3e, chunks %.3e" % (rms["streamed"], rms["chunks"]), flush=True)
    assert rms["streamed"] <= 1.1 * rms["chunks"]
