"""Performance cases of the KV-cached semantic operators.

Each case is one thing a program does with this library through its public calls: evaluating
a filter, a map or a mixed batch over cached documents, building the caches (plainly or with
compression scores), selecting a compressed profile, and fitting, training and running the
proxy.  Sizes are those of the scale workload (the d_model 2048 decoder, documents of
lognormal length around 512 tokens, 32-token suffixes, the retention grid, the 2048 -> 256
proxy at batch 512); single decoder blocks are that decoder with two layers.

Inputs come from the seed alone.  Document lengths are the quantiles of their distribution, so
that the work of a case depends on the case and not on the seed.
"""
import math
import statistics

import numpy as np
import torch

from paper_2602_04430_amd import kvop as K
from paper_2602_04430_amd import synth

D_MODEL, HEADS, KV_HEADS, HEAD_DIM, D_FFN, VOCAB = 2048, 16, 8, 128, 5632, 32000
STD = 0.02
LABEL_LO, LABEL_N = synth.MAP_SLICE
DTYPES = {
    "f32": (K.KVOP_F32, K.KVOP_KV_F32, 4),
    "bf16": (K.KVOP_BF16, K.KVOP_KV_BF16, 2),
    "fp8": (K.KVOP_BF16, K.KVOP_KV_FP8, 1),
}


def listed():
    return [
        # one document of median length through the whole decoder: the latency of a single answer
        {"name": "filter_one", "kind": "filter", "layers": 16, "cache": "bf16", "docs": 1, "median": 512, "suffix": 32,
         "r": 1.0},
        # a collection of about a thousand documents, whole decoder: the throughput of a filter
        {"name": "filter_many", "kind": "filter", "layers": 16, "cache": "bf16", "docs": 1024, "median": 512,
         "suffix": 32, "r": 1.0},
        # a compressed profile over an FP8 cache: the cheap stages of a cascade
        {"name": "filter_fp8", "kind": "filter", "layers": 2, "cache": "fp8", "docs": 512, "median": 512, "suffix": 32,
         "r": 0.25},
        # the plain FP32 form, the precision baseline that BF16 answers are compared with
        {"name": "filter_fp32", "kind": "filter", "layers": 2, "cache": "f32", "docs": 64, "median": 512, "suffix": 32,
         "r": 1.0},
        # a map: eight greedily decoded ids per document, mostly single-row decoding steps
        {"name": "map", "kind": "map", "layers": 2, "cache": "bf16", "docs": 192, "median": 384, "suffix": 32, "r": 1.0},
        # filter, map and join items sharing one pass (a third of the documents each)
        {"name": "mixed", "kind": "mixed", "layers": 2, "cache": "bf16", "docs": 768, "median": 384, "suffix": 32,
         "r": 1.0},
        # new documents arrive: caches and pooled features are built, a filter answers, the caches go
        {"name": "ingest", "kind": "ingest", "layers": 2, "cache": "bf16", "docs": 128, "median": 512, "suffix": 32,
         "r": 1.0},
        # offline build that also scores every row for the compressed profiles
        {"name": "scored_build", "kind": "scored", "layers": 2, "cache": "bf16", "docs": 96, "median": 512,
         "suffix": 32},
        # the retained lists of one compressed profile of the scale collection
        {"name": "select", "kind": "select", "docs": 4096, "median": 512, "r": 0.25},
        # start of proxy training: the standardiser over all training rows, the first minibatch
        {"name": "proxy_fit", "kind": "fit", "rows": 20000, "d_in": 2048, "hidden": 256, "batch": 512},
        # one minibatch of proxy training: forward and backward
        {"name": "proxy_grads", "kind": "grads", "rows": 20000, "d_in": 2048, "hidden": 256, "batch": 512},
        # the proxy as first stage over a collection of fresh documents
        {"name": "proxy_infer", "kind": "infer", "rows": 20000, "d_in": 2048, "hidden": 256, "tau": 0.9},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["filter", "filter", "filter", "map", "mixed", "ingest", "scored", "select", "fit", "grads",
                       "infer"])
    if kind in ("fit", "grads", "infer"):
        case = {"kind": kind, "rows": _log(rng, 513, 20000), "d_in": rng.choice([1024, 2048]),
                "hidden": rng.choice([128, 256])}
        if kind == "infer":
            case["rows"] = _log(rng, 1, 20000)
            case["tau"] = rng.choice([0.9, 0.95, 0.99])
        else:
            case["batch"] = 8 * _log(rng, 8, 64)
        return case
    if kind == "select":
        return {"kind": kind, "docs": _log(rng, 1, 4096), "median": rng.randint(128, 512),
                "r": rng.choice([0.5, 0.25, 0.1])}
    median, suffix = rng.randint(100, 512), rng.randint(9, 48)
    if kind == "filter":
        cache = rng.choice(["bf16", "bf16", "fp8", "f32"])
        layers = 16 if cache != "f32" and rng.random() < 0.4 else 2
        most = 64 if cache == "f32" else 512
        return {"kind": kind, "layers": layers, "cache": cache, "docs": _log(rng, 1, most), "median": median,
                "suffix": suffix, "r": rng.choice([1.0, 0.5, 0.25, 0.1])}
    case = {"kind": kind, "layers": 2, "cache": rng.choice(["bf16", "fp8"]), "median": median, "suffix": suffix}
    if kind == "scored":
        case["docs"] = _log(rng, 1, 96)
    else:
        case["docs"] = _log(rng, 3, {"map": 192, "mixed": 768, "ingest": 128}[kind])
        case["r"] = 1.0 if kind == "ingest" else rng.choice([1.0, 0.5])
    return case


# ----------------------------------------------------------------------------- sizes


def _lengths(case):
    """Quantiles of lognormal(ln median, 1), clipped to [16, 8 median], in a scattered order."""
    n, med = case["docs"], case["median"]
    z = statistics.NormalDist()
    q = [min(max(int(round(med * math.exp(z.inv_cdf((i + 0.5) / n)))), 16), 8 * med) for i in range(n)]
    step = max(1, int(n * 0.618))
    while math.gcd(step, n) != 1:
        step += 1
    return [q[(i * step) % n] for i in range(n)]


def _kept(case, lengths):
    return [synth.retained_count(case.get("r", 1.0), n) for n in lengths]


def _thirds(n):
    """Documents of a mixed batch: filter items, map items, join pairs."""
    pairs = n // 6
    maps = (n - 2 * pairs) // 2
    return n - 2 * pairs - maps, maps, pairs


def _items(case, keys):
    """(cached keys, decoded ids) of every item the case evaluates."""
    if case["kind"] == "map":
        return [(k, synth.MAP_TOKENS) for k in keys]
    if case["kind"] == "mixed":
        f, m, p = _thirds(len(keys))
        side = keys[f + m:]
        return ([(k, 1) for k in keys[:f]] + [(k, synth.MAP_TOKENS) for k in keys[f:f + m]] +
                [(side[2 * i] + side[2 * i + 1], 1) for i in range(p)])
    return [(k, 1) for k in keys]


def _row_flops(c):
    """Projections of one row of one layer: queries, keys and values, output with the feed-forward."""
    q = 2 * D_MODEL * HEADS * HEAD_DIM
    kv = 2 * D_MODEL * 2 * KV_HEADS * HEAD_DIM
    return q, kv, q + 6 * D_MODEL * D_FFN


def _weight_bytes(case, layers):
    q, kv, rest = _row_flops(case)
    return layers * (q + kv + rest) // 2 * (4 if case["cache"] == "f32" else 2)


def _op_work(case, keys):
    q, kv, rest = _row_flops(case)
    S, NL = case["suffix"], case["layers"]
    per_key = 2 * KV_HEADS * HEAD_DIM * DTYPES[case["cache"]][2]
    att = 4 * HEADS * HEAD_DIM
    flops, read = 0, _weight_bytes(case, NL)
    for k, ids in _items(case, keys):
        rows = S * (NL - 1) + 1                       # the last layer continues with the last row only
        flops += rows * rest + S * (NL - 2) * (q + kv) + S * kv + q   # layer 0's projection is shared
        flops += att * (S * (NL - 1) + 1) * k
        read += NL * k * per_key * ids
        flops += (ids - 1) * NL * (q + kv + rest + att * (k + S))
        if ids > 1:
            flops += ids * 2 * D_MODEL * LABEL_N
    return {"bytes": read, "flops": flops}


def _build_work(case, lengths):
    q, kv, rest = _row_flops(case)
    NL, rows = case["layers"], sum(lengths)
    keys = sum(n * (n + 1) // 2 for n in lengths)
    return {"bytes": _weight_bytes(case, NL) + rows * (NL * 2 * KV_HEADS * HEAD_DIM * DTYPES[case["cache"]][2] + 2 * D_MODEL),
            "flops": NL * (rows * (q + kv + rest) + 4 * HEADS * HEAD_DIM * keys)}


def work(case):
    kind = case["kind"]
    if kind == "select":
        n = sum(_lengths(case))
        return {"bytes": 4 * (n + sum(_kept(case, _lengths(case)))), "flops": n}
    if kind in ("fit", "grads", "infer"):
        d, h = case["d_in"], case["hidden"]
        if kind == "infer":
            return {"bytes": case["rows"] * (4 * d + 6) + 2 * d * h, "flops": 2 * case["rows"] * (d * h + 2 * h)}
        b = case["batch"]
        w = {"bytes": 4 * b * d + 2 * d * h + 4 * d * h, "flops": 4 * b * d * h}
        if kind == "fit":
            w["bytes"] += 4 * case["rows"] * d
            w["flops"] += 4 * case["rows"] * d
        return w
    lengths = _lengths(case)
    if kind == "scored":
        w = _build_work(case, lengths)
        # per row, layer and query head: the query covariance and the key's quadratic form
        w["flops"] += sum(lengths) * case["layers"] * HEADS * 4 * HEAD_DIM * HEAD_DIM
        return w
    w = _op_work(case, _kept(case, lengths))
    if kind == "ingest":
        b = _build_work(case, lengths)
        w = {k: w[k] + b[k] for k in w}
    return w


# ----------------------------------------------------------------------------- inputs


def _generator(seed, stream):
    return torch.Generator(device="cuda").manual_seed((int(seed) * 64 + stream) % (1 << 62))


def _shape(case):
    return synth.ModelShape(case["layers"], D_MODEL, HEADS, KV_HEADS, HEAD_DIM, D_FFN, VOCAB)


def _weights(case, seed):
    """Packed FP32 master weights: matrices N(0, 0.02^2), norm gains near 1."""
    shape = _shape(case)
    flat = torch.randn(shape.numel(), generator=_generator(seed, 0), device="cuda").mul_(STD)
    at = 0
    for name, shp in synth.weight_order(shape):
        n = math.prod(shp)
        if name.endswith("norm"):
            flat[at:at + n] += 1.0
        at += n
    return flat


def _tokens(case, seed):
    n = sum(_lengths(case))
    return torch.randint(0, VOCAB, (n,), generator=_generator(seed, 1), device="cuda", dtype=torch.int32)


def _suffixes(case, seed):
    rng = np.random.default_rng([int(seed), 2])
    return [rng.integers(0, VOCAB, case["suffix"]).astype(np.int32) for _ in range(3)]


def _lists(case, lengths, seed):
    """Retained rows of every document: the first four, the rest at random; ascending."""
    rng = np.random.default_rng([int(seed), 3])
    out, offs = [], [0]
    for n, k in zip(lengths, _kept(case, lengths)):
        if k == n:
            out.append(np.arange(n, dtype=np.int32))
        else:
            h = min(4, n)
            rest = rng.permutation(n - h)[:k - h] + h
            out.append(np.concatenate([np.arange(h), np.sort(rest)]).astype(np.int32))
        offs.append(offs[-1] + k)
    return np.concatenate(out), np.asarray(offs, np.int64)


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int64)


class _State(dict):
    """What a program keeps: library objects go when it goes."""

    def __del__(self):
        torch.cuda.synchronize()
        for key, drop in (("pool", K.kvop_pool_destroy), ("model", K.kvop_model_destroy),
                          ("proxy", K.kvop_proxy_destroy)):
            if self.get(key) is not None:
                drop(self[key])


def _model_state(case, seed):
    s = _State(case=case)
    compute, kv, _ = DTYPES[case["cache"]]
    s["model"] = K.kvop_model_create(K.make_cfg(_shape(case)), _weights(case, seed), compute)
    lengths = _lengths(case)
    per_row = 2 * case["layers"] * KV_HEADS * HEAD_DIM * DTYPES[case["cache"]][2]
    size = sum(n * per_row + (case["layers"] * KV_HEADS * 8 * ((n + 15) // 16) if case["cache"] == "fp8" else 0) + 512
               for n in lengths)
    s["pool"] = K.kvop_pool_create(s["model"], kv, size)
    s["offsets"] = _offsets(lengths)
    s["tokens"] = _tokens(case, seed)
    return s


def _op(case, kind, suffix):
    if kind == K.KVOP_MAP:
        return K.make_op(kind, suffix, label_lo=LABEL_LO, label_n=LABEL_N, n_gen=synth.MAP_TOKENS)
    return K.make_op(kind, suffix, synth.YES_ID, synth.NO_ID)


def _answers(n):
    return {"logits": torch.empty(n, 2, device="cuda"), "decision": torch.empty(n, dtype=torch.int8, device="cuda")}


def _texts(n):
    return {"logits": torch.empty(n, synth.MAP_TOKENS, LABEL_N, device="cuda"),
            "ids": torch.empty(n, synth.MAP_TOKENS, dtype=torch.int32, device="cuda")}


def _features(case, seed):
    """Pooled document features: every dimension with its own mean and spread."""
    g = _generator(seed, 4)
    d = case["d_in"]
    mean = torch.randn(d, generator=g, device="cuda")
    std = torch.rand(d, generator=g, device="cuda").add_(0.1)
    feats = torch.randn(case["rows"], d, generator=g, device="cuda").mul_(std).add_(mean)
    return feats, mean, 1.0 / std


def _proxy_params(case, seed):
    h, d = case["hidden"], case["d_in"]
    return torch.randn(h * d + 3 * h + 2, generator=_generator(seed, 5), device="cuda").mul_(STD)


def _minibatch(case, seed):
    g = _generator(seed, 6)
    labels = torch.randint(0, 2, (case["rows"],), generator=g, device="cuda", dtype=torch.int32)
    rows = torch.randperm(case["rows"], generator=g, device="cuda")[:case["batch"]].to(torch.int32)
    return labels, rows


def _scores(case, seed):
    """Expected-attention scores of every row: positive, heavy-tailed."""
    n = sum(_lengths(case))
    return torch.randn(n, generator=_generator(seed, 7), device="cuda").exp_().mul_(0.05)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "select":
        s = _State(case=case)
        tiny = synth.TINY
        s["model"] = K.kvop_model_create(K.make_cfg(tiny), torch.zeros(tiny.numel(), device="cuda"), K.KVOP_BF16)
        s["pool"] = K.kvop_pool_create(s["model"], K.KVOP_KV_BF16, 1 << 20)
        s["offsets"] = _offsets(_lengths(case))
        s["scores"] = _scores(case, seed)
        s["idx"] = torch.empty(sum(_kept(case, _lengths(case))), dtype=torch.int32, device="cuda")
        return s
    if kind in ("fit", "grads", "infer"):
        s = _State(case=case)
        s["proxy"] = K.kvop_proxy_create(case["d_in"], case["hidden"], _proxy_params(case, seed))
        s["feats"], mean, istd = _features(case, seed)
        if kind != "fit":
            K.kvop_proxy_set_standardizer(s["proxy"], mean, istd)
            torch.cuda.synchronize()
        n = case["rows"]
        if kind == "infer":
            s["cls"] = torch.empty(n, dtype=torch.int8, device="cuda")
            s["conf"] = torch.empty(n, device="cuda")
            s["answered"] = torch.empty(n, dtype=torch.int8, device="cuda")
        else:
            s["labels"], s["rows"] = _minibatch(case, seed)
            s["grads"] = torch.empty(case["hidden"] * case["d_in"] + 3 * case["hidden"] + 2, device="cuda")
            s["loss"] = torch.empty(1, device="cuda")
        return s
    s = _model_state(case, seed)
    lengths, n = _lengths(case), case["docs"]
    if kind == "scored":
        s["scores"] = torch.empty(sum(lengths), device="cuda")
        s["pooled"] = torch.empty(n, D_MODEL, device="cuda")
        return s
    idx, s["list_offsets"] = _lists(case, lengths, seed)
    s["idx"] = torch.from_numpy(idx).cuda()
    sf = _suffixes(case, seed)
    s["op"] = _op(case, K.KVOP_MAP if kind == "map" else K.KVOP_FILTER, sf[0])
    s["out"] = _texts(n) if kind == "map" else _answers(n)
    if kind == "ingest":
        s["pooled"] = torch.empty(n, D_MODEL, device="cuda")
        return s
    s["handles"] = K.kvop_kv_build(s["pool"], s["tokens"], s["offsets"])
    if kind == "mixed":
        f, m, p = _thirds(n)
        s["out"] = {"filter": _answers(f), "map": _texts(m), "join": _answers(p)}
        ops = [_op(case, k, sf[i]) for i, k in enumerate((K.KVOP_FILTER, K.KVOP_MAP, K.KVOP_JOIN))]
        o = s["out"]
        s["ops"] = [(ops[0], o["filter"]["logits"], o["filter"]["decision"], None),
                    (ops[1], o["map"]["logits"], None, o["map"]["ids"]),
                    (ops[2], o["join"]["logits"], o["join"]["decision"], None)]
        s["item_op"] = np.asarray([0] * f + [1] * m + [2] * p, np.int32)
        s["item_list"] = np.asarray(list(range(f + m)) + [f + m + 2 * i for i in range(p)], np.int64)
    return s


# ----------------------------------------------------------------------------- the pass


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "filter":
        K.kvop_op_eval(s["pool"], s["op"], case["r"], s["idx"], s["list_offsets"], s["handles"], s["out"]["logits"],
                       s["out"]["decision"])
        return s["out"]
    if kind == "map":
        K.kvop_op_eval(s["pool"], s["op"], case["r"], s["idx"], s["list_offsets"], s["handles"], s["out"]["logits"],
                       None, s["out"]["ids"])
        return s["out"]
    if kind == "mixed":
        K.kvop_mixed_eval(s["pool"], s["ops"], case["r"], s["idx"], s["list_offsets"], s["handles"], s["item_op"],
                          s["item_list"], 0)
        return s["out"]
    if kind == "ingest":
        handles = K.kvop_kv_build(s["pool"], s["tokens"], s["offsets"], s["pooled"])
        K.kvop_op_eval(s["pool"], s["op"], case["r"], s["idx"], s["list_offsets"], handles, s["out"]["logits"],
                       s["out"]["decision"])
        K.kvop_kv_release(s["pool"], handles)
        return {"pooled": s["pooled"], **s["out"]}
    if kind == "scored":
        handles = K.kvop_kv_build_scored(s["pool"], s["tokens"], s["offsets"], case["suffix"], s["scores"], s["pooled"])
        K.kvop_kv_release(s["pool"], handles)
        return {"scores": s["scores"], "pooled": s["pooled"]}
    if kind == "select":
        offsets = K.kvop_ea_select(s["pool"], s["scores"], s["offsets"], case["r"], s["idx"])
        return {"idx": s["idx"], "offsets": offsets}
    if kind == "infer":
        K.kvop_proxy_infer(s["proxy"], s["feats"], case["tau"], s["cls"], s["conf"], s["answered"])
        return {"cls": s["cls"], "conf": s["conf"], "answered": s["answered"]}
    if kind == "fit":
        K.kvop_proxy_fit_standardizer(s["proxy"], s["feats"])
    K.kvop_proxy_grads(s["proxy"], s["feats"], s["labels"], s["rows"], case["batch"], s["grads"], s["loss"])
    return {"grads": s["grads"], "loss": s["loss"]}


# ----------------------------------------------------------------------------- 64-bit values


def _norm(x, g):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + 1e-5) * g


def _rotate(x, pos):
    half = HEAD_DIM // 2
    inv = 10000.0 ** (-2.0 * torch.arange(half, device=x.device, dtype=torch.float64) / HEAD_DIM)
    a = pos.double()[:, None] * inv
    c, s = a.cos()[:, None, :], a.sin()[:, None, :]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], -1)


class _Exact:
    """The decoder in 64 bits, one document or item at a time."""

    def __init__(self, case, seed):
        flat, at, self.w = _weights(case, seed), 0, {}
        for name, shp in synth.weight_order(_shape(case)):
            n = math.prod(shp)
            self.w[name] = flat[at:at + n].view(shp).double()
            at += n
        self.layers = case["layers"]

    def attend(self, q, k, v, mask):
        g = HEADS // KV_HEADS
        q = q.transpose(0, 1).reshape(KV_HEADS, g * q.shape[0], HEAD_DIM)
        sc = q.contiguous() @ k.permute(1, 2, 0).contiguous() / math.sqrt(HEAD_DIM)
        if mask is not None:
            sc = sc.view(KV_HEADS, g, *mask.shape).masked_fill(~mask, -math.inf).view_as(sc)
        o = sc.softmax(-1) @ v.transpose(0, 1).contiguous()
        return o.view(KV_HEADS * g, -1, HEAD_DIM).transpose(0, 1).reshape(-1, HEADS * HEAD_DIM)

    def qkv(self, l, x):
        h = _norm(x, self.w[f"L{l}.attn_norm"])
        return (h @ self.w[f"L{l}.{n}"].T for n in ("wq", "wk", "wv"))

    def rest(self, l, x, o):
        x = x + o @ self.w[f"L{l}.wo"].T
        h = _norm(x, self.w[f"L{l}.ffn_norm"])
        f = torch.nn.functional.silu(h @ self.w[f"L{l}.w_gate"].T) * (h @ self.w[f"L{l}.w_up"].T)
        return x + f @ self.w[f"L{l}.w_down"].T

    def build(self, tokens, scores=None, n_future=0):
        """Rotated keys and values of every layer, and the final hidden rows."""
        x = self.w["embed"][tokens.long()]
        n = len(tokens)
        pos = torch.arange(n, device=x.device)
        mask = pos[:, None] >= pos[None, :]
        cache = []
        for l in range(self.layers):
            q, k, v = self.qkv(l, x)
            q, k, v = q.view(n, HEADS, -1), _rotate(k.view(n, KV_HEADS, -1), pos), v.view(n, KV_HEADS, -1)
            if scores is not None:
                scores += self.expected(q, k, v, n_future)
            cache.append((k, v))
            x = self.rest(l, x, self.attend(_rotate(q, pos), k, v, mask))
        return cache, x

    def expected(self, q, k, v, n_future):
        """Every row's share of one layer's expected attention by queries just after the document."""
        n, half = q.shape[0], HEAD_DIM // 2
        eye = torch.eye(HEAD_DIM, device=q.device, dtype=torch.float64)
        fut = torch.arange(n, n + n_future, device=q.device)
        R = _rotate(eye[None].expand(n_future, -1, -1), fut).mean(0).T
        mu = q.mean(0)
        qc = (q - mu).transpose(0, 1)
        cov = R @ (qc.transpose(1, 2) @ qc / n) @ R.T
        mu = mu @ R.T
        g = HEADS // KV_HEADS
        kk = k.transpose(0, 1).repeat_interleave(g, 0)
        e = (kk @ mu[:, :, None])[..., 0] / math.sqrt(HEAD_DIM) + ((kk @ cov) * kk).sum(-1) / (2 * HEAD_DIM)
        c = e.softmax(-1).view(KV_HEADS, g, n).mean(1) * v.norm(dim=-1).T
        return (c / c.sum(-1, keepdim=True)).sum(0)

    def answer(self, suffix, docs, ids=None):
        """Hidden last row of a suffix over cached documents [(cache, kept rows, length)], then
        one more for each id of `ids` that is fed back."""
        dev = suffix.device
        own = [([], []) for _ in range(self.layers)]
        pos0, out = sum(d[2] for d in docs), []
        for tok in [suffix] + [ids[i:i + 1] for i in range(len(ids) if ids is not None else 0)]:
            x, n = self.w["embed"][tok.long()], len(tok)
            pos = torch.arange(pos0, pos0 + n, device=dev)
            for l in range(self.layers):
                q, k, v = self.qkv(l, x)
                q = q.view(n, HEADS, -1)
                own[l][0].append(_rotate(k.view(n, KV_HEADS, -1), pos))
                own[l][1].append(v.view(n, KV_HEADS, -1))
                ks, vs, before = [], [], 0
                for cache, kept, length in docs:
                    # document B's rows sit after document A: its keys move by A's length
                    kb = cache[l][0][kept]
                    ks.append(kb if before == 0 else _rotate(kb, torch.full((len(kept),), before, device=dev)))
                    vs.append(cache[l][1][kept])
                    before += length
                ks, vs = torch.cat(ks + own[l][0]), torch.cat(vs + own[l][1])
                mask = None
                if n > 1:
                    mask = torch.ones(n, len(ks), dtype=torch.bool, device=dev)
                    mask[:, len(ks) - n:] = torch.ones(n, n, dtype=torch.bool, device=dev).tril()
                x = self.rest(l, x, self.attend(_rotate(q, pos), ks, vs, mask))
            pos0 += n
            out.append(_norm(x[-1], self.w["final_norm"]))
        return torch.stack(out)


def _exact_ops(case, seed):
    """Logits in 64 bits; a map's later steps follow its own ids, so only its first has a value."""
    ex = _Exact(case, seed)
    lengths, tokens = _lengths(case), _tokens(case, seed)
    offs = _offsets(lengths)
    idx, lo = _lists(case, lengths, seed)
    suffixes = [torch.from_numpy(s).cuda() for s in _suffixes(case, seed)]
    head = ex.w["head"]
    pair = head[[synth.YES_ID, synth.NO_ID]]
    pooled = []

    def doc(i):
        cache, x = ex.build(tokens[offs[i]:offs[i + 1]])
        if case["kind"] == "ingest":
            pooled.append(_norm(x, ex.w["final_norm"]).mean(0))
        return cache, torch.from_numpy(idx[lo[i]:lo[i + 1]]).cuda().long(), lengths[i]

    def answers(suffix, items):
        return {"logits": torch.stack([pair @ ex.answer(suffix, [doc(i) for i in it])[0] for it in items]),
                "decision": None}

    n = case["docs"]
    if case["kind"] == "mixed":
        f, m, p = _thirds(n)
        return {"filter": answers(suffixes[0], [[i] for i in range(f)]), "map": {"logits": None, "ids": None},
                "join": answers(suffixes[2], [[f + m + 2 * i, f + m + 2 * i + 1] for i in range(p)])}
    out = answers(suffixes[0], [[i] for i in range(n)])
    return {"pooled": torch.stack(pooled), **out} if case["kind"] == "ingest" else out


def _exact_scored(case, seed):
    ex = _Exact(case, seed)
    lengths, tokens = _lengths(case), _tokens(case, seed)
    offs, scores, pooled = _offsets(lengths), [], []
    for i, n in enumerate(lengths):
        sc = torch.zeros(n, device="cuda", dtype=torch.float64)
        _, x = ex.build(tokens[offs[i]:offs[i + 1]], sc, case["suffix"])
        scores.append(sc)
        pooled.append(_norm(x, ex.w["final_norm"]).mean(0))
    return {"scores": torch.cat(scores), "pooled": torch.stack(pooled)}


def _exact_proxy(case, seed):
    d, h = case["d_in"], case["hidden"]
    p = _proxy_params(case, seed).double().requires_grad_(case["kind"] != "infer")
    feats, mean, istd = _features(case, seed)
    if case["kind"] == "fit":
        x = feats.double()
        mean, istd = x.mean(0), 1.0 / x.std(0, correction=0).clamp_min(1e-6)
    w1, b1 = p[:h * d].view(h, d), p[h * d:h * d + h]
    w2, b2 = p[h * d + h:h * d + 3 * h].view(2, h), p[h * d + 3 * h:]

    def logits(x):
        x = (x.double() - mean.double()) * istd.double()
        return torch.nn.functional.gelu(x @ w1.T + b1) @ w2.T + b2

    if case["kind"] == "infer":
        return {"cls": None, "conf": logits(feats).softmax(-1).max(-1).values, "answered": None}
    labels, rows = _minibatch(case, seed)
    loss = torch.nn.functional.cross_entropy(logits(feats[rows.long()]), labels[rows.long()].long())
    loss.backward()
    return {"grads": p.grad, "loss": loss.detach().view(1)}


def exact(case, seed):
    kind = case["kind"]
    if kind == "select":
        return None                       # whole numbers only
    if kind in ("fit", "grads", "infer"):
        return _exact_proxy(case, seed)
    if case["layers"] * sum(_lengths(case)) > 1500000 or kind == "map":
        return None                       # too long in 64 bits; a map's ids decide its later logits
    if case["layers"] > 2 and case["docs"] < 8:
        return None                       # a few logits of a deep 16-bit model: rounding decides their norm
    if kind == "scored":
        return _exact_scored(case, seed)
    return _exact_ops(case, seed)
