"""What this library's users have it do, as cases that can be timed and compared.

Every case goes through the package's own entry points: `DecodeLayer` (one decode step of an attention layer, or its
attention alone), `ChunkSelector` (a chunk of prompt tokens) and nothing below them.  Inputs are drawn on the GPU from
the seed, after the recipe of workloads.py: Q, K, V ~ N(0, 1), and for every query head a share of the tokens is
critical, its key pushed towards that head's query; pages are a random permutation of the pool.
"""
import math
import random

import numpy as np
import torch

from paper_2411_02886_amd import binding as ts
from paper_2411_02886_amd.runtime import ChunkSelector, DecodeLayer

_DEV = "cuda:0"
_DTYPES = {"f32": (ts.TS_F32, torch.float32, 4), "bf16": (ts.TS_BF16, torch.bfloat16, 2)}


def _case(kind, dtype, B, n_lo, n_hi, H, H_kv, D, k, P=16, C=1, n_init=0, n_local=0, planted=0.005, beta=2.5, steps=1,
          name=None):
    c = dict(kind=kind, dtype=dtype, B=B, n_lo=n_lo, n_hi=n_hi, H=H, H_kv=H_kv, D=D, k=k, P=P, C=C, n_init=n_init,
             n_local=n_local, planted=planted, beta=beta, steps=steps)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer: one short fp32 sequence, where launches and latency are all there is
        _case("step", "f32", 1, 4096, 4096, 8, 2, 64, 256, planted=0.0078, beta=3.0, name="step_4k_fp32"),
        # one long conversation, one decode step of one layer (32 query heads over 8 KV heads)
        _case("step", "bf16", 1, 131072, 131072, 32, 8, 128, 2048, name="step_128k"),
        # the longest context: one decode step over a million cached tokens (28 over 4), few critical tokens
        _case("step", "bf16", 1, 1048576, 1048576, 28, 4, 128, 4096, planted=0.001, name="step_1m"),
        # a server's batch of conversations of very different lengths, none of them a round number
        _case("step", "bf16", 32, 1031, 16001, 32, 8, 128, 2048, name="step_batch32"),
        # wide layer (eight query heads per KV head, 8 KV heads), the paper's page size of 1 and its forced blocks
        _case("step", "bf16", 4, 20011, 40009, 64, 8, 128, 2048, P=1, n_init=128, n_local=512, name="step_wide_page1"),
        # eight consecutive decode steps of eight sequences with the Selection Cache at the paper's threshold
        _case("cached", "bf16", 8, 16384, 65536, 32, 8, 128, 2048, steps=8, name="cached_run_8x8"),
        # attention over a selection that is already there (every layer step that hits the cache): a large batch ...
        _case("attend", "bf16", 64, 3001, 9001, 32, 8, 128, 2048, name="attend_batch64"),
        # ... and seven query heads per KV head, longer selections
        _case("attend", "bf16", 48, 8191, 12289, 28, 4, 128, 4096, n_init=128, n_local=512, name="attend_batch48_g7"),
        # prefill: selection for a chunk of 512 queries over a quarter of a million cached tokens
        _case("chunk_select", "bf16", 1, 262144, 262144, 32, 8, 128, 4096, C=512, name="chunk_select_256k"),
        # the same for two prompts at once, ragged lengths, a ragged chunk and the forced blocks (28 over 4)
        _case("chunk_select", "bf16", 2, 12007, 30011, 28, 4, 128, 2048, C=300, n_init=128, n_local=512,
              name="chunk_select_ragged"),
        # prefill: the chunk's attention over its selection and itself
        _case("chunk_attend", "bf16", 1, 65536, 65536, 32, 8, 128, 4096, C=512, name="chunk_attend_512"),
        # prefill as the paper prints it: one selection per chunk with the mean query, then the attention
        _case("chunk_mean", "bf16", 1, 131072, 131072, 32, 8, 128, 4096, C=512, name="chunk_mean_128k"),
    ]


_HEADS = [(8, 2, 64), (32, 8, 128), (28, 4, 128), (32, 4, 128), (64, 8, 128), (16, 16, 64), (24, 8, 64), (40, 8, 128),
          (12, 2, 128), (32, 8, 64)]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "cached", "attend", "attend", "chunk_select", "chunk_attend", "chunk_mean"])
    H, H_kv, D = rng.choice(_HEADS)
    P = rng.choice([16, 16, 16, 32, 1])
    k = _log(rng, 256, 4096)
    n_init, n_local = rng.choice([(0, 0), (0, 0), (128, 512), (4, 61)])
    dtype = "bf16"
    C = steps = 1
    if kind == "step":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        B = rng.choice([1, 1, 1, 2, 5, 16, 32])
        n_hi = min(_log(rng, 2000, 600000), 400000 // B, (1 << 28) // (H_kv * D * B))
    elif kind == "cached":
        B, steps = rng.choice([1, 3, 8]), rng.randint(4, 8)
        n_hi = min(_log(rng, 4000, 65536), 300000 // B)
    elif kind == "attend":
        B = _log(rng, 1, 96)
        n_hi = rng.randint(k, 3 * k + 1000)
    else:
        C = rng.choice([64, 128, 300, 512, 777])
        B = rng.choice([1, 1, 2, 3])
        n_hi = _log(rng, 4000, 200000)
        if kind == "chunk_select":
            n_hi = max(2000, min(n_hi, (1 << 31) // (B * C * H)))
        else:
            n_hi = max(2000, n_hi // (2 * B))
    n_lo = rng.randint(max(1, n_hi // 3), n_hi)
    n_lo, n_hi = n_lo - (n_lo + 1) % 2 if n_lo > 1 else n_lo, n_hi
    return _case(kind, dtype, B, n_lo, n_hi, H, H_kv, D, k, P=P, C=C, n_init=n_init, n_local=n_local, steps=steps)


# ---------------------------------------------------------------------------------------------------------------------

def _lengths(c):
    """Cached tokens of every sequence (the chunk's own tokens come on top of them)."""
    r = random.Random(1000003 * c["n_lo"] + 10007 * c["n_hi"] + c["B"])
    return [r.randint(c["n_lo"], c["n_hi"]) for _ in range(c["B"])]


def _inputs(c, seed):
    """Queries [steps][B][C][H][D], pools and page table; all values made from the seed."""
    tdt = _DTYPES[c["dtype"]][1]
    g = torch.Generator(device=_DEV).manual_seed(int(seed) * 7919 + 17)
    B, C, H, H_kv, D, P = c["B"], c["C"], c["H"], c["H_kv"], c["D"], c["P"]
    cached = _lengths(c)
    lens = [n + (C if C > 1 else 0) for n in cached]
    pages = [(n + P - 1) // P for n in lens]
    indptr = np.concatenate([[0], np.cumsum(pages)]).astype(np.int32)
    perm = torch.randperm(int(indptr[-1]), generator=g, device=_DEV)
    shape = (int(indptr[-1]), P, H_kv, D)
    k_pool = torch.empty(shape, dtype=tdt, device=_DEV).normal_(generator=g)
    v_pool = torch.empty(shape, dtype=tdt, device=_DEV).normal_(generator=g)
    q = [torch.randn((B, C, H, D), generator=g, device=_DEV)]
    for _ in range(c["steps"] - 1):     # consecutive queries of a conversation resemble each other
        q.append(0.95 * q[-1] + math.sqrt(1.0 - 0.95 ** 2) * torch.randn((B, C, H, D), generator=g, device=_DEV))
    flat = k_pool.view(-1, H_kv, D)
    kv = (torch.arange(H, device=_DEV) // (H // H_kv))[:, None]
    for b in range(B):
        npl = int(round(c["planted"] * cached[b]))
        if npl == 0 or c["beta"] == 0.0:
            continue
        pos = torch.randperm(cached[b], generator=g, device=_DEV)[:npl * H].view(H, npl)
        slot = perm[int(indptr[b]) + pos // P] * P + pos % P
        u = q[0][b].permute(1, 0, 2)                                    # [H][C][D]
        u = c["beta"] * u / u.norm(dim=-1, keepdim=True)
        u = u[:, torch.arange(npl, device=_DEV) % C]                    # the j-th planted token serves query j mod C
        flat[slot, kv] = (flat[slot, kv].float() + u).to(tdt)
    return dict(q=[x.to(tdt) for x in q], k_pool=k_pool, v_pool=v_pool, indptr=indptr, perm=perm, lens=lens, cached=cached)


def _some_selection(c, x, seed):
    """A selection as a previous step left it: k ascending tokens of every sequence, -1 behind its count."""
    g = torch.Generator(device=_DEV).manual_seed(int(seed) * 104729 + 5)
    idx = torch.full((c["B"], c["k"]), -1, dtype=torch.int32, device=_DEV)
    count = torch.zeros((c["B"],), dtype=torch.int32, device=_DEV)
    for b, n in enumerate(x["cached"]):
        lo = min(c["n_init"], n)
        hi = max(lo, n - c["n_local"])
        m = min(c["k"], hi - lo)
        idx[b, :m] = (lo + torch.randperm(hi - lo, generator=g, device=_DEV)[:m].sort().values).int()
        count[b] = m
    return idx, count


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    bits = torch.int16 if c["dtype"] == "bf16" else torch.float32
    common = dict(H=c["H"], H_kv=c["H_kv"], D=c["D"], P=c["P"], k=c["k"], k_pool=x["k_pool"].view(bits),
                  v_pool=x["v_pool"].view(bits), page_indptr=x["indptr"], page_indices=x["perm"].cpu().numpy(),
                  seq_lens=x["lens"], num_initial=c["n_init"], num_local=c["n_local"])
    if c["C"] > 1:
        layer = ChunkSelector(C=c["C"], **common)
    else:
        layer = DecodeLayer(dtype=_DTYPES[c["dtype"]][0], **common)
    if c["kind"] in ("attend", "chunk_attend"):
        layer.idx, layer.count = _some_selection(c, x, seed)
    return dict(kind=c["kind"], layer=layer, q=[q.view(bits) for q in x["q"]], sm=1.0 / math.sqrt(c["D"]),
                bf16=c["dtype"] == "bf16")


def run(state):
    layer, q, kind = state["layer"], state["q"], state["kind"]
    if kind == "step":                      # one decode step, in the form that the layer says is the faster one
        layer.step(q[0], compact=None, ranked_vote=True)
    elif kind == "cached":                  # a new conversation's first steps: nothing cached before the first
        layer.first.fill_(1)
        for qt in q:
            layer.step(qt, theta=0.9, compact=None, ranked_vote=True)
    elif kind in ("attend", "chunk_attend"):
        layer.attend(q[0], state["sm"])
    elif kind == "chunk_select":
        layer.select(q[0])
        # the index set as marks on the tokens (a cache manager's view of it): two tokens that change places at the
        # end of the ranking are two marks, whereas in the ascending list they move every entry between them
        kept = torch.zeros(layer.votes.shape, dtype=torch.uint8, device=layer.votes.device)
        kept.scatter_(1, layer.idx.clamp(min=0).long(), 1)
        return dict(votes=layer.votes, kept=kept, count=layer.count)
    else:
        layer.select_mean_query(q[0])
        layer.attend(q[0], state["sm"])
    out = layer.out.view(torch.bfloat16) if state["bf16"] else layer.out
    if kind in ("attend", "chunk_attend"):
        return dict(out=out, lse=layer.lse)
    return dict(out=out, lse=layer.lse, idx=layer.idx, count=layer.count)


def work(case):
    """K is read once by a selection, K and V of the selected tokens once by the attention; the chunk form's softmax
    needs every product of Q and K once."""
    c = case
    es, row = _DTYPES[c["dtype"]][2], c["H_kv"] * c["D"] * _DTYPES[c["dtype"]][2]
    n = sum(_lengths(c))
    att = sum(min(m, c["k"] + c["n_init"] + c["n_local"]) for m in _lengths(c))
    own = c["B"] * c["C"] if c["C"] > 1 else 0
    qo = 2 * c["B"] * c["C"] * c["H"] * c["D"] * es
    hd = c["H"] * c["D"]
    att_bytes = 2 * (att + own) * row + qo + (att + own) * 4
    att_flops = 4.0 * c["C"] * hd * (att + own / 2)
    if c["kind"] in ("attend", "chunk_attend"):
        return dict(bytes=att_bytes, flops=att_flops)
    if c["kind"] == "chunk_select":
        return dict(bytes=n * row + qo / 2 + n * 4, flops=2.0 * c["C"] * hd * n)
    if c["kind"] == "chunk_mean":
        return dict(bytes=n * row + qo / 2 + att_bytes, flops=2.0 * hd * n + att_flops)
    if c["kind"] == "cached":
        # the first step selects; whether a later one does is in the data: each attends
        return dict(bytes=n * row + c["steps"] * att_bytes, flops=2.0 * hd * n + c["steps"] * att_flops)
    return dict(bytes=n * row + att_bytes, flops=2.0 * hd * n + att_flops)


def tolerance(case):
    # whole values: two tokens whose votes agree to the rounding of the scores may change places
    if case["kind"] == "chunk_select":
        return {"rel": 2e-5, "max": 1e-4, "differ": 0.001}      # float votes, sums over thousands of rows
    if case["dtype"] == "bf16":
        return {"rel": 1e-2, "max": 0.1, "differ": 0.01}        # bf16 outputs
    return {"rel": 1e-5, "max": 1e-4, "differ": 0.01}           # float outputs


# ---------------------------------------------------------------------------------------------------------------------
# the same in 64 bits

def _logical(c, x, pool, b, pos):
    """Rows of logical tokens `pos` of sequence b as doubles: [len][H_kv][D]."""
    slot = x["perm"][int(x["indptr"][b]) + pos // c["P"]] * c["P"] + pos % c["P"]
    return pool.view(-1, c["H_kv"], c["D"])[slot].double()


def _scores(c, qb, rows):
    """[C][H][len] products of qb [C][H][D] (double) with rows [len][H_kv][D]."""
    C, G = qb.shape[0], c["H"] // c["H_kv"]
    out = torch.empty((C, c["H"], rows.shape[0]), dtype=torch.float64, device=_DEV)
    for kv in range(c["H_kv"]):
        qs = qb[:, kv * G:(kv + 1) * G].reshape(C * G, c["D"])
        out[:, kv * G:(kv + 1) * G] = (qs @ rows[:, kv].t().contiguous()).view(C, G, -1)
    return out


def _ranked(c, n):
    lo = min(c["n_init"], n)
    return lo, max(lo, n - c["n_local"])


def _votes(c, x, b, qb):
    """Soft votes of all cached tokens for the queries qb [C][H][D]: summed over heads and queries."""
    n = x["cached"][b]
    lo, hi = _ranked(c, n)
    votes = torch.zeros(n, dtype=torch.float64, device=_DEV)
    if hi <= lo:
        return votes
    step = max(1024, (1 << 26) // max(1, qb.shape[0] * c["H"]))
    lse = None
    for sweep in (0, 1):
        for t in range(lo, hi, step):
            pos = torch.arange(t, min(hi, t + step), device=_DEV)
            s = _scores(c, qb, _logical(c, x, x["k_pool"], b, pos))
            if sweep == 0:
                part = torch.logsumexp(s, dim=2)
                lse = part if lse is None else torch.logaddexp(lse, part)
            else:
                votes[pos] = torch.exp(s - lse[:, :, None]).sum(dim=(0, 1))
    return votes


def _select(c, x, b, qb):
    n = x["cached"][b]
    lo, hi = _ranked(c, n)
    k = min(c["k"], hi - lo)
    v = _votes(c, x, b, qb)
    return lo + torch.topk(v[lo:hi], k).indices.sort().values


def _attend(c, x, b, qb, sel):
    """Joint softmax over the forced tokens, the selected ones and, in a chunk, its own tokens so far."""
    n, C, G = x["cached"][b], c["C"], c["H"] // c["H_kv"]
    lo, hi = _ranked(c, n)
    own = torch.arange(n, n + C, device=_DEV) if C > 1 else torch.arange(0, device=_DEV)
    pos = torch.cat([torch.arange(lo, device=_DEV), sel.long(), torch.arange(hi, n, device=_DEV), own])
    s = _scores(c, qb, _logical(c, x, x["k_pool"], b, pos)) / math.sqrt(c["D"])
    if C > 1:
        hidden = own[None, :] - n > torch.arange(C, device=_DEV)[:, None]
        s[:, :, pos.numel() - C:].masked_fill_(hidden[:, None, :], -math.inf)
    lse = torch.logsumexp(s, dim=2)
    p = torch.exp(s - lse[:, :, None])
    v = _logical(c, x, x["v_pool"], b, pos)
    out = torch.empty((C, c["H"], c["D"]), dtype=torch.float64, device=_DEV)
    for kv in range(c["H_kv"]):
        ps = p[:, kv * G:(kv + 1) * G].reshape(C * G, -1)
        out[:, kv * G:(kv + 1) * G] = (ps @ v[:, kv].contiguous()).view(C, G, -1)
    return out, lse


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    if c["kind"] == "cached":
        return None                         # which steps select is a decision of its own: the step cases are exact
    B = c["B"]
    q = x["q"][0].double()
    if c["kind"] == "chunk_select":
        votes = torch.zeros((B, max(x["lens"])), dtype=torch.float64, device=_DEV)
        for b in range(B):
            votes[b, :x["cached"][b]] = _votes(c, x, b, q[b])
        return dict(votes=votes, kept=None, count=None)
    if c["kind"] in ("attend", "chunk_attend"):
        idx, count = _some_selection(c, x, seed)
        sel = [idx[b, :int(count[b])] for b in range(B)]
    elif c["kind"] == "chunk_mean":
        mean = q.mean(dim=1, keepdim=True).float().to(torch.bfloat16).double()
        sel = [_select(c, x, b, mean[b]) for b in range(B)]
    else:
        sel = [_select(c, x, b, q[b]) for b in range(B)]
    got = [_attend(c, x, b, q[b], sel[b]) for b in range(B)]
    return dict(out=torch.stack([o for o, _ in got]), lse=torch.stack([l for _, l in got]), idx=None, count=None)
