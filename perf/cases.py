"""The work that users of this framework have it do, as cases that can be timed
and compared.

A case is one of four kinds of pass, each through the public entry points of
``paper_2608_05483_amd.plora``:

  call    one projection of one batch, called eagerly: ``segment_apply``
          (grouping and LoRA apply).  Prompt batches, mixed batches and the
          smallest calls.
  step    the LoRA work of one decode step over several layers, captured once
          as a HIP graph and replayed, as serving engines run decode: the
          grouping with the first projection (``segment_apply``), then per
          layer the projections that share the layer's input in one call
          (``apply_multi``: q, k, v) and the output projection (``apply``).
  split   the rank-reduced intermediate taken apart from the expansion (the
          form that ships v between devices): ``segment``, ``shrink``,
          ``expand``.
  attn    split-KV decode attention of one layer: ``attn_decode``.

The adapter populations, widths, ranks and id distributions are those of
``paper_2608_05483_amd/workloads.py``, ``bench.py`` and the tests.  The outputs
y accumulate in place, as the entry points define them, so a pass on the same
state adds the same delta again.
"""
import math

import numpy as np
import torch

from paper_2608_05483_amd import plora as P

DEV = "cuda"


def listed():
    return [
        # the smallest call there is: one projection of a small model, eager
        # (latency and launch overhead)
        dict(name="tiny_call", kind="call", T=8, h_in=256, h_out=256, N=4, ranks="8",
             ids="uniform", requests=0, none=0.0),
        # one user's token through eight 7B-shaped layers
        dict(name="decode_one", kind="step", T=1, layers=8, h=4096, h_kv=4096, N=1000,
             ranks="16", ids="zipf", alpha=1.0, none=0.0),
        # the benchmark's decode batch (64 requests over 1000 skewed adapters of
        # rank 16) through four 7B-shaped layers
        dict(name="decode_64", kind="step", T=64, layers=4, h=4096, h_kv=4096, N=1000,
             ranks="16", ids="zipf", alpha=1.0, none=0.0),
        # a grouped-query layer pair at the largest ranks, ragged batch, a tenth of
        # the requests on the base model
        dict(name="decode_gqa_r128", kind="step", T=45, layers=2, h=8192, h_kv=1024, N=300,
             ranks="64,128", ids="uniform", alpha=0.0, none=0.1),
        # ranks that users do train and that are no multiple of 8, 13B widths
        dict(name="decode_odd_ranks", kind="step", T=100, layers=2, h=5120, h_kv=5120, N=200,
             ranks="4,6,10,12,20,40", ids="zipf", alpha=0.8, none=0.0),
        # the largest decode batch, every request on its own rank-64 adapter
        dict(name="decode_256_r64", kind="step", T=256, layers=1, h=4096, h_kv=4096, N=1000,
             ranks="64", ids="uniform", alpha=0.0, none=0.0),
        # speculative or chunked decoding over ragged ranks, 13B widths
        dict(name="ragged_512", kind="call", T=512, h_in=5120, h_out=5120, N=1000,
             ranks="8,16,32,64", ids="zipf", alpha=0.8, requests=0, none=0.05),
        # prompts of 1..512 tokens of 32 requests mixed in one batch, into a
        # grouped-query k/v projection
        dict(name="prefill_kv", kind="call", T=8317, h_in=8192, h_out=1024, N=1000,
             ranks="32", ids="uniform", requests=32, none=0.0),
        # few long prompts, the largest batch the entry points take
        dict(name="prefill_long", kind="call", T=16384, h_in=4096, h_out=4096, N=200,
             ranks="16,64", ids="uniform", requests=7, none=0.0),
        # the shipped intermediate, ragged batch
        dict(name="split_700", kind="split", T=700, h_in=4096, h_out=4096, N=500,
             ranks="32", ids="zipf", alpha=1.0, requests=0, none=0.0),
        # decode attention of a full batch (the benchmark's shape)
        dict(name="attn_batch", kind="attn", batch=64, heads=32, max_len=4096, min_len=512),
        # decode attention of a few long contexts on a head-parallel shard
        dict(name="attn_few_long", kind="attn", batch=3, heads=8, max_len=30011, min_len=9000),
    ]


RANK_SETS = ("8", "16", "32", "64", "8,16,32,64", "8,16,32,64,128", "4,8,16", "6,12,20",
             "64,128", "16,64")


def _loguni(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _width(rng, lo, hi):
    """A model width: a multiple of 8, mostly of 128."""
    w = _loguni(rng, lo, hi)
    return max(lo, w // 128 * 128 if rng.random() < 0.7 else w // 8 * 8)


def _ids(rng):
    return rng.choice([dict(ids="uniform", alpha=0.0), dict(ids="zipf", alpha=1.0),
                       dict(ids="zipf", alpha=0.8)])


def _fit(N, per_adapter, most):
    """An adapter count whose stacks take at most ``most`` bytes."""
    return max(1, min(N, int(most // per_adapter)))


def draw(rng):
    kind = rng.choice(["step", "step", "call", "call", "split", "attn"])
    if kind == "attn":
        heads = rng.choice([4, 8, 16, 32])
        batch = _loguni(rng, 1, 64)
        max_len = _loguni(rng, 64, min(32768, 64 * 32 * 4096 // (heads * batch)))
        return dict(kind="attn", batch=batch, heads=heads, max_len=max_len,
                    min_len=rng.randint(1, max_len))
    ranks = rng.choice(RANK_SETS)
    top = max(int(r) for r in ranks.split(","))
    none = rng.choice([0.0, 0.0, 0.1])
    N = _loguni(rng, 4, 1000)
    if kind == "step":
        layers = rng.randint(1, 3)
        h = _width(rng, 1024, 8192)
        h_kv = h if rng.random() < 0.5 else max(512, h // 8 // 8 * 8)
        per = 2.0 * top * layers * (2 * (2 * h) + 2 * (h + h_kv))
        return dict(kind="step", T=_loguni(rng, 1, 256), layers=layers, h=h, h_kv=h_kv,
                    N=_fit(N, per, 5e9), ranks=ranks, none=none, **_ids(rng))
    h_in, h_out = _width(rng, 512, 8192), _width(rng, 512, 8192)
    T = _loguni(rng, 4, 8192)
    T = max(4, min(T, int(1.5e8 // (h_in + 2 * h_out))))
    c = dict(kind=kind, T=T, h_in=h_in, h_out=h_out,
             N=_fit(N, 2.0 * top * (h_in + h_out), 3e9), ranks=ranks, none=none, **_ids(rng))
    # long batches are mostly prompts: runs of tokens of one adapter
    c["requests"] = rng.randint(1, 40) if T > 256 and rng.random() < 0.7 else 0
    return c


# ---- inputs ----------------------------------------------------------------------


def _rank_list(case):
    return [int(r) for r in case["ranks"].split(",")]


def _probs(case):
    N = case["N"]
    if case["ids"] == "zipf":
        w = np.arange(1, N + 1, dtype=np.float64) ** -case["alpha"]
        return w / w.sum()
    return np.full(N, 1.0 / N)


def _request_lengths(case):
    """Lengths of the case's requests: part of the case, not of the seed."""
    T, n = case["T"], min(case["requests"], case["T"])
    w = np.random.default_rng(T * 64 + n).random(n) + 0.01
    lens = np.maximum(1, np.floor(w / w.sum() * T)).astype(np.int64)
    while lens.sum() > T:
        lens[lens.argmax()] -= 1
    lens[lens.argmin()] += T - lens.sum()
    return lens


def _token_ids(case, rng):
    N, T = case["N"], case["T"]
    n = case.get("requests") or T
    if case.get("requests"):
        lens = _request_lengths(case)
        n = len(lens)
    ids = rng.choice(N, size=n, p=_probs(case)).astype(np.int32)
    if case["none"]:
        ids[rng.random(n) < case["none"]] = -1
    return np.repeat(ids, lens).astype(np.int32) if case.get("requests") else ids


def _normal(shape, std, gen):
    return torch.empty(shape, dtype=torch.bfloat16, device=DEV).normal_(0.0, std, generator=gen)


def _stack(case, h_in, h_out, ranks, gen):
    """One projection's adapters: A_i and B_i blocks back to back, scaled so
    that a token's delta has about the size of the base output."""
    r = ranks.astype(np.int64)
    a_off = np.concatenate([[0], np.cumsum(r * h_in)[:-1]])
    b_off = np.concatenate([[0], np.cumsum(r * h_out)[:-1]])
    A = _normal(int((r * h_in).sum()), h_in ** -0.5, gen)
    B = _normal(int((r * h_out).sum()), float(r.mean()) ** -0.5, gen)
    scales = torch.tensor([0.5, 1.0, 2.0], device=DEV)[
        torch.randint(0, 3, (case["N"],), device=DEV, generator=gen)]
    top = int(max(_rank_list(case)))
    return P.Adapters(A, B, torch.from_numpy(a_off).to(DEV), torch.from_numpy(b_off).to(DEV),
                      torch.from_numpy(ranks).to(DEV), scales, h_in, h_out,
                      max(8, (top + 7) // 8 * 8))


def _ranks(case, rng):
    rl = np.asarray(_rank_list(case), np.int32)
    return rl[rng.integers(0, len(rl), case["N"])]


class State:
    pass


def _lora_state(case, seed):
    """Everything a LoRA case has in hand before its pass."""
    s = State()
    s.case = case
    rng = np.random.default_rng([seed, 17])
    gen = torch.Generator(device=DEV).manual_seed(seed)
    T, N = case["T"], case["N"]
    s.idx = torch.from_numpy(_token_ids(case, rng)).to(DEV)
    s.segs = P.Segments(T, N, device=DEV)
    # unused entries of the grouping stay as allocated where nothing writes them
    for t in (s.segs.perm, s.segs.seg_ptr, s.segs.seg_id, s.segs.tiles):
        t.zero_()
    ranks = _ranks(case, rng)
    if case["kind"] == "step":
        h, kv = case["h"], case["h_kv"]
        s.layers = []
        for _ in range(case["layers"]):
            x, xo = _normal((T, h), 1.0, gen), _normal((T, h), 1.0, gen)
            ads = [_stack(case, h, w, ranks, gen) for w in (h, kv, kv, h)]
            ys = [_normal((T, w), 1.0, gen) for w in (h, kv, kv, h)]
            s.layers.append((x, xo, ads, ys))
        s.ws = P.Workspace(T, s.layers[0][2][:3], device=DEV)
    else:
        s.x = _normal((T, case["h_in"]), 1.0, gen)
        s.ad = _stack(case, case["h_in"], case["h_out"], ranks, gen)
        s.y = _normal((T, case["h_out"]), 1.0, gen)
        s.ws = P.Workspace(T, s.ad, device=DEV)
        if case["kind"] == "split":
            s.v = torch.zeros((T, s.ad.max_rank), dtype=torch.float32, device=DEV)
    return s


def _step_calls(s):
    """The calls of one decode step."""
    for i, (x, xo, ads, ys) in enumerate(s.layers):
        if i == 0:
            P.segment_apply(s.idx, x, ads[0], s.segs, ys[0], s.ws)
            P.apply_multi(x, ads[1:3], s.segs, ys[1:3], s.ws)
        else:
            P.apply_multi(x, ads[:3], s.segs, ys[:3], s.ws)
        P.apply(xo, ads[3], s.segs, ys[3], s.ws)


def _attn_lens(case, seed):
    rng = np.random.default_rng([seed, 19])
    # stratified over [min_len, max_len], so that every seed reads about as much
    lo, hi, b = case["min_len"], case["max_len"], case["batch"]
    u = (rng.permutation(b) + rng.random(b)) / b
    return np.minimum(hi, np.floor(lo + u * (hi + 1 - lo))).astype(np.int32)


def prepare(case, seed):
    if case["kind"] == "attn":
        s = State()
        s.case = case
        gen = torch.Generator(device=DEV).manual_seed(seed)
        b, h, n = case["batch"], case["heads"], case["max_len"]
        s.q = _normal((b, h, P.ATTN_HEAD_DIM), 1.0, gen)
        s.k = _normal((b, h, n, P.ATTN_HEAD_DIM), 1.0, gen)
        s.v = _normal((b, h, n, P.ATTN_HEAD_DIM), 1.0, gen)
        s.lens = torch.from_numpy(_attn_lens(case, seed)).to(DEV)
        s.out = torch.zeros((b, h, P.ATTN_HEAD_DIM), dtype=torch.bfloat16, device=DEV)
        s.ws = torch.empty(P.attn_workspace_bytes(b, h, n), dtype=torch.uint8, device=DEV)
        s.scale = P.ATTN_HEAD_DIM ** -0.5
        return s
    s = _lora_state(case, seed)
    if case["kind"] == "step":
        # one eager step first (kernels are loaded outside the capture), then the
        # graph; the outputs go back to the base projections' values
        keep = [[y.clone() for y in layer[3]] for layer in s.layers]
        _step_calls(s)
        s.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(s.graph):
            _step_calls(s)
        for layer, ys in zip(s.layers, keep):
            for y, k in zip(layer[3], ys):
                y.copy_(k)
    return s


# ---- one pass ----------------------------------------------------------------------


def _grouping(segs):
    return {"perm": segs.perm, "seg_ptr": segs.seg_ptr, "seg_id": segs.seg_id,
            "meta": segs.meta, "tiles": segs.tiles}


def run(s):
    kind = s.case["kind"]
    if kind == "attn":
        P.attn_decode(s.q, s.k, s.v, s.lens, s.scale, s.out, s.ws)
        return {"out": s.out}
    if kind == "step":
        s.graph.replay()
        return {"y": [y for layer in s.layers for y in layer[3]], "seg": _grouping(s.segs)}
    if kind == "split":
        P.segment(s.idx, s.segs, ws=s.ws)
        P.shrink(s.x, s.ad, s.segs, s.v, s.ws)
        P.expand(s.v, s.ad, s.segs, s.y)
        return {"v": s.v, "y": s.y, "seg": _grouping(s.segs)}
    P.segment_apply(s.idx, s.x, s.ad, s.segs, s.y, s.ws)
    return {"y": s.y, "seg": _grouping(s.segs)}


def _projections(case):
    """(h_in, h_out) of every projection of a pass, and the distinct inputs."""
    if case["kind"] == "step":
        h, kv = case["h"], case["h_kv"]
        return [(h, h), (h, kv), (h, kv), (h, h)] * case["layers"], [h, h] * case["layers"]
    return [(case["h_in"], case["h_out"])], [case["h_in"]]


def work(case):
    """Bytes: every distinct adapter's A_i and B_i, x and the ids read once, y
    read and written once (v written and read once where it is shipped); keys
    and values of every valid position.  Counts that depend on the draw are the
    expected ones."""
    if case["kind"] == "attn":
        keys = case["batch"] * case["heads"] * 0.5 * (case["min_len"] + case["max_len"])
        d = P.ATTN_HEAD_DIM
        return {"bytes": keys * d * 4 + case["batch"] * case["heads"] * d * 4,
                "flops": keys * d * 4}
    T = case["T"]
    live = 1.0 - case["none"]
    n = (min(case["requests"], T) if case.get("requests") else T) * live
    distinct = float(np.sum(1.0 - (1.0 - _probs(case)) ** n))
    r = float(np.mean(_rank_list(case)))
    projections, inputs = _projections(case)
    b = 4.0 * T + sum(2.0 * T * live * h for h in inputs)
    f = 0.0
    for h_in, h_out in projections:
        b += 2.0 * r * (h_in + h_out) * distinct + 4.0 * T * live * h_out
        f += 2.0 * T * live * r * (h_in + h_out)
    if case["kind"] == "split":
        b += 8.0 * T * live * r
    return {"bytes": b, "flops": f}


def tolerance(case):
    """bf16 outputs of fp32 sums, rounded once: another order of the sums moves
    a value to its neighbour now and then.  Against the 64-bit result rounded
    once, the outputs are up to 1e-4 off in norm and one bf16 step (0.0078) in
    a value; the stated bounds are four times the first, and a step for each of
    two passes on one state with room for the scale of the difference.  The
    grouping is whole numbers."""
    return {"rel": 4e-4, "max": 0.02}


# ---- the same in 64 bits ------------------------------------------------------------


def _exact_delta(x, ad, idx, ranks, a_off, b_off, y):
    """(v, y + s (x A_i) B_i) in float64, adapter by adapter."""
    out = y.double()
    v = torch.zeros((x.shape[0], ad.max_rank), dtype=torch.float64, device=DEV)
    for i in np.unique(idx[idx >= 0]):
        tok = torch.from_numpy(np.flatnonzero(idx == i)).to(DEV)
        r = int(ranks[i])
        A = ad.A[a_off[i]:a_off[i] + ad.h_in * r].view(ad.h_in, r).double()
        B = ad.B[b_off[i]:b_off[i] + ad.h_out * r].view(r, ad.h_out).double()
        m = x[tok].double() @ A
        v[tok, :r] = m
        out[tok] += ad.scales[int(i)].double() * (m @ B)
    return v, out


def exact(case, seed):
    if case["kind"] == "attn":
        s = prepare(case, seed)
        out = torch.zeros(s.out.shape, dtype=torch.float64, device=DEV)
        for b, n in enumerate(s.lens.tolist()):
            for h in range(case["heads"]):
                w = (s.k[b, h, :n].double() * s.q[b, h].double()).sum(1) * s.scale
                w = torch.softmax(w, 0)
                out[b, h] = (w[:, None] * s.v[b, h, :n].double()).sum(0)
        return {"out": out}
    s = _lora_state(case, seed)
    idx = s.idx.cpu().numpy()
    none = {"perm": None, "seg_ptr": None, "seg_id": None, "meta": None, "tiles": None}
    if case["kind"] == "step":
        ys = []
        for x, xo, ads, outs in s.layers:
            for p, (ad, y) in enumerate(zip(ads, outs)):
                meta = [t.cpu().numpy() for t in (ad.ranks, ad.a_off, ad.b_off)]
                ys.append(_exact_delta(x if p < 3 else xo, ad, idx, *meta, y)[1])
        return {"y": ys, "seg": none}
    meta = [t.cpu().numpy() for t in (s.ad.ranks, s.ad.a_off, s.ad.b_off)]
    v, y = _exact_delta(s.x, s.ad, idx, *meta, s.y)
    if case["kind"] == "split":
        return {"v": v, "y": y, "seg": none}
    return {"y": y, "seg": none}
