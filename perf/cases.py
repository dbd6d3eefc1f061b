"""The calls whose speed is followed, as programs that use this framework make them.

A program compresses a reasoning model's KV cache at step boundaries (score,
select and compact), decodes tokens over the retained cache (a whole cache per
call, or one layer per call inside a captured graph, or through the decoder
loop), draws each token from the penalised logits and probes the answer's
perplexity.  The listed cases are those calls at the shapes of the workloads
in `inputs.WORKLOADS`; `draw` takes them over the ranges around those shapes:
1 to 28 layers, 1 to 32 sequences of 256 to 65,536 rows (even or ragged),
2 to 8 KV heads with groups of 2 to 8 query heads, head_dim 64 and 128, bf16
and fp32, windows of 8 to 128 tokens, 1 to 256 logit rows of 4,096 to 152,064
tokens.
"""
import math

import numpy as np
import torch

from paper_2608_04771_amd import binding as B
from paper_2608_04771_amd import inputs as I
from paper_2608_04771_amd.controller import RecoDecoder, RecoPolicy

TAUS_BETAS = (0.4, 0.8, 0.0, 1.0, 3.0)      # reward bands and their penalties (RecoPolicy's defaults)


def _decode(name, layers, batch, hq, hkv, dim, dtype, lo, hi, append, graph=False):
    return {"name": name, "kind": "decode", "layers": layers, "batch": batch, "hq": hq, "hkv": hkv, "dim": dim,
            "dtype": dtype, "lo": lo, "hi": hi, "append": append, "graph": graph}


def _score(name, layers, batch, hq, hkv, dim, dtype, lo, hi, w, fed, causal=True):
    return {"name": name, "kind": "score", "layers": layers, "batch": batch, "hq": hq, "hkv": hkv, "dim": dim,
            "dtype": dtype, "lo": lo, "hi": hi, "w": w, "fed": fed, "causal": causal}


def _select(name, layers, batch, hkv, dim, dtype, lo, hi, w, r_lo, r_hi, pool=1):
    return {"name": name, "kind": "select", "layers": layers, "batch": batch, "hkv": hkv, "dim": dim, "dtype": dtype,
            "lo": lo, "hi": hi, "w": w, "r_lo": r_lo, "r_hi": r_hi, "pool": pool}


def _sample(name, rows, vocab, ids, temperature):
    return {"name": name, "kind": "sample", "rows": rows, "vocab": vocab, "ids": ids, "temperature": temperature}


def _ppl(name, batch, n, vocab):
    return {"name": name, "kind": "ppl", "batch": batch, "n": n, "vocab": vocab}


def listed():
    return [
        # The smallest call: one layer of a small fp32 model attending over 2,048 rows.
        _decode("decode_f32_small", 1, 1, 8, 2, 64, "f32", 2048, 2048, False),
        # A model's decode step: 28 per-layer calls in one captured graph, one 7B-shaped sequence after compression.
        _decode("decode_step_graph_7b", 28, 1, 28, 4, 128, "bf16", 9645, 9645, True, graph=True),
        # The same cache in one call over all layers.
        _decode("decode_all_layers_7b", 28, 1, 28, 4, 128, "bf16", 9645, 9645, True),
        # One layer of a serving batch: 32 ragged sequences.
        _decode("decode_layer_batch32", 1, 32, 28, 4, 128, "bf16", 4096, 32768, True),
        # The largest decode: many long units (8 layers of the 32B shape, 8 sequences).
        _decode("decode_32b", 8, 8, 40, 8, 128, "bf16", 24577, 24577, True),
        # Compression of the 7B-shaped 16K cache: two-pass scoring, then selection and compaction.
        _score("score_7b_16k", 28, 1, 28, 4, 128, "bf16", 16384, 16384, 64, False),
        _select("select_compact_7b_16k", 28, 1, 4, 128, "bf16", 16384, 16384, 64, 0.5808, 0.5808),
        # Long caches scored in one pass with the decode statistics of the window tokens (32B shape, 2 layers).
        _score("score_fed_32b_64k", 2, 4, 40, 8, 128, "bf16", 65536, 65536, 32, True),
        # The smallest compression: a small fp32 model's 2,048 rows.
        _score("score_f32_small", 1, 1, 8, 2, 64, "f32", 2048, 2048, 32, False),
        # The draws of 256 generated tokens over a 152,064-token vocabulary, penalty fused.
        _sample("sample_256_rows", 256, 152064, 64, 1.0),
        # The answer probe of one sequence: 32 answer tokens.
        _ppl("answer_ppl_7b", 1, 32, 152064),
        # One reasoning step of the decoder loop on the 8B shape: compress at the boundary, then 256 tokens, each
        # decoded over about 1.1K rows of all layers and drawn from its penalised 128,256-token row.
        {"name": "loop_step_8b", "kind": "loop", "layers": 32, "batch": 1, "hq": 32, "hkv": 8, "dim": 128,
         "dtype": "bf16", "lo": 993, "hi": 993, "w": 32, "tokens": 256, "vocab": 128256, "reward": 0.41},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng, max_elems):
    """Layers, sequences, heads and a row range whose K (or V) holds at most max_elems elements."""
    hkv, group = rng.choice([(2, 4), (4, 7), (8, 4), (8, 5), (4, 8), (8, 2)])
    dim = 128 if rng.random() < 0.75 else 64
    dtype = "bf16" if rng.random() < 0.8 else "f32"
    while True:
        layers, batch = _log_int(rng, 1, 28), _log_int(rng, 1, 32)
        hi = _log_int(rng, 256, 65536)
        lo = hi if rng.random() < 0.5 else max(256, int(hi * rng.uniform(0.1, 0.9)))
        if layers * batch * hkv * hi * dim <= max_elems:
            return layers, batch, hkv, group, dim, dtype, lo, hi


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "score", "score", "select", "sample", "ppl"])
    if kind == "decode":
        layers, batch, hkv, group, dim, dtype, lo, hi = _draw_shape(rng, 1.0e9)
        c = _decode("", layers, batch, hkv * group, hkv, dim, dtype, lo, hi, rng.random() < 0.75, rng.random() < 0.25)
    elif kind == "score":
        while True:
            layers, batch, hkv, group, dim, dtype, lo, hi = _draw_shape(rng, 3.0e8)
            w = rng.choice([8, 16, 31, 32, 64, 100, 128])
            # fp32 products run at a sixteenth of the bf16 rate
            if layers * batch * hkv * hi * dim * 2.0 * group * w <= (2.0e11 if dtype == "bf16" else 1.2e10):
                break
        fed = rng.random() < 0.4
        c = _score("", layers, batch, hkv * group, hkv, dim, dtype, lo, hi, w, fed, fed or rng.random() < 0.8)
    elif kind == "select":
        layers, batch, hkv, group, dim, dtype, lo, hi = _draw_shape(rng, 5.0e8)
        r_hi = round(rng.uniform(0.3, 1.0), 3)
        c = _select("", layers, batch, hkv, dim, dtype, lo, hi, rng.choice([16, 32, 64]),
                    round(rng.uniform(0.2, r_hi), 3), r_hi, rng.choice([1, 1, 1, 5, 7]))
    else:
        vocab = rng.choice([4096, 32000, 50001, 128256, 151931, 152064])
        if kind == "sample":
            c = _sample("", _log_int(rng, 1, 256), vocab, rng.choice([1, 64, 300]), rng.choice([0.0, 0.6, 1.0, 1.0]))
        else:
            c = _ppl("", _log_int(rng, 1, 8), _log_int(rng, 4, 32), vocab)
    del c["name"]
    return c


# ------------------------------------------------------------------ inputs
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _lens(case):
    """The rows of every sequence: spread evenly over [lo, hi], in a mixed order."""
    n = case["batch"]
    x = np.round(np.linspace(case["lo"], case["hi"], n)).astype(np.int64)
    return np.random.RandomState(5).permutation(x)


def _elem(case):
    return 4 if case["dtype"] == "f32" else 2


def _cache(case, seed, hq, w, slack):
    """Cache, window queries and generator of `case`, drawn as the workloads' are."""
    lens = _lens(case)
    wl = I.Workload("case", case["layers"], case["batch"], hq, case["hkv"], case["dim"], case["dtype"],
                    tuple(int(x) for x in lens), w, 0, "beta22", int(seed))
    ci = I.make_cache(wl, device=_device(), capacity=int(lens.max()) + slack, seq_lens=lens)
    return wl, ci


def _scale(case):
    return 1.0 / math.sqrt(case["dim"])


def _decode_inputs(case, seed):
    wl, ci = _cache(case, seed, case["hq"], 1, 64)
    q, kn, vn = (x[0] for x in I.make_decode_inputs(wl, ci, 1, device=_device()))
    return ci, q, kn, vn


def _stats64(case, ci):
    """(max, sum) of every window row's log2-domain logits, as the window tokens' decode steps report them."""
    NL, Bs, hkv, G, w = case["layers"], case["batch"], case["hkv"], case["hq"] // case["hkv"], case["w"]
    st = torch.zeros((NL, Bs, case["hq"], w, 2), dtype=torch.float64, device=ci.k.device)
    for l in range(NL):
        for b in range(Bs):
            n = int(ci.seq_len[b])
            for h in range(hkv):
                x = _logits64(case, ci.k[l, b, h, :n], ci.q_win[l, b, h * G:(h + 1) * G], True)
                m = x.amax(-1)
                st[l, b, h * G:(h + 1) * G, :, 0] = m * math.log2(math.e)
                st[l, b, h * G:(h + 1) * G, :, 1] = torch.exp(x - m[..., None]).sum(-1)
    return st


def _logits64(case, k, q, causal):
    """Scaled fp64 logits [G][w][n] of window queries q [G][w][D] over keys k [n][D] (-inf: not visible)."""
    n, w = k.shape[0], q.shape[1]
    x = torch.matmul(q.double().reshape(-1, q.shape[2]), k.double().T.contiguous()).reshape(q.shape[0], w, n)
    x = x * _scale(case)
    if causal:
        pos = torch.arange(n - w, n, device=k.device)
        x = x.masked_fill(torch.arange(n, device=k.device)[None, None, :] > pos[None, :, None], -math.inf)
    return x


def _loop_inputs(case, seed):
    """Prompt cache, prompt window queries, and one step's queries, K/V rows, logit rows and reflection ids."""
    wl, ci = _cache(case, seed, case["hq"], case["w"], 2 * case["tokens"] + 64)
    qs, ks, vs = I.make_decode_inputs(wl, ci, case["tokens"], device=_device())
    logits = I.make_logits(0, 0, seed + 17, device=_device(), shape=(case["tokens"], case["batch"], case["vocab"]))
    ids = torch.from_numpy(I.make_reflection_ids(64, case["vocab"], 1003)).to(_device())
    return ci, qs, ks, vs, logits, ids


def prepare(case, seed):
    kind = case["kind"]
    dev = _device()
    if kind == "decode":
        ci, q, kn, vn = _decode_inputs(case, seed)
        cache = B.KVCache(ci.k, ci.v, ci.length)
        out = torch.empty_like(q)
        lse = torch.empty(q.shape[:3], dtype=torch.float32, device=dev)
        if not case["append"]:
            kn = vn = None
        err = torch.zeros(1, dtype=torch.int32, device=dev)
        s = {"kind": kind, "cache": cache, "q": q, "kn": kn, "vn": vn, "out": out, "lse": lse, "graph": None}
        if not case["graph"]:
            # the form a decoder loop keeps: buffers checked once, one call per token
            s["call"] = B.PreparedDecode(cache, case["hq"], out, lse, B.decode_workspace(cache, case["hq"]), err)
            return s
        ws = B.decode_workspace(cache, case["hq"], 1)

        def step():
            for l in range(case["layers"]):
                B.reco_decode_attn(cache, q[l:l + 1], None if kn is None else kn[l:l + 1],
                                   None if vn is None else vn[l:l + 1], out=out[l:l + 1], lse=lse[l:l + 1],
                                   layer0=l, n_layers=1, ws=ws, dev_err=err)
            if kn is not None:
                cache.length.sub_(1)

        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):
            step()
        torch.cuda.current_stream().wait_stream(side)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            step()
        s["graph"], s["ws"], s["err"] = graph, ws, err
        return s
    if kind == "score":
        wl, ci = _cache(case, seed, case["hq"], case["w"], 64)
        cache = B.KVCache(ci.k, ci.v, ci.length)
        stats = _stats64(case, ci).float() if case["fed"] else None
        return {"kind": kind, "case": case, "cache": cache, "q": ci.q_win, "stats": stats,
                "scores": torch.zeros(ci.k.shape[:4], dtype=torch.float32, device=dev),
                "ws": torch.empty(B.score_workspace_size(cache, case["hq"], case["w"]), dtype=torch.uint8, device=dev)}
    if kind == "select":
        wl, ci = _cache(case, seed, case["hkv"], 1, 64)
        cache = B.KVCache(ci.k, ci.v, ci.length)
        g = torch.Generator(device=dev)
        g.manual_seed(int(seed) + 23)
        # attention mass is close to lognormal over the keys
        scores = torch.exp(torch.randn(ci.k.shape[:4], generator=g, device=dev, dtype=torch.float32)) * 1e-2
        r = np.linspace(case["r_lo"], case["r_hi"], case["batch"])
        return {"kind": kind, "case": case, "cache": cache, "scores": scores, "full": ci.length.clone(),
                "r": torch.from_numpy(r).to(dev), "kept": torch.zeros(ci.k.shape[:4], dtype=torch.int32, device=dev),
                "pooled": torch.zeros_like(scores) if case["pool"] > 1 else None,
                "ws": torch.empty(B.select_compact_workspace_size(cache), dtype=torch.uint8, device=dev)}
    if kind == "sample":
        rows, vocab = case["rows"], case["vocab"]
        logits = I.make_logits(rows, vocab, int(seed), device=dev)
        ids = torch.from_numpy(I.make_reflection_ids(case["ids"], vocab, 1001)).to(dev)
        reward = torch.from_numpy(I.make_rewards("beta22", rows, 1, int(seed))[:, 0].copy()).to(dev)
        ws = torch.empty(B.penalty_sample_workspace_size(rows, vocab), dtype=torch.uint8, device=dev)
        tokens = torch.empty(rows, dtype=torch.int32, device=dev)
        return {"kind": kind, "case": case, "logits": logits, "seed": int(seed),
                "call": B.PreparedPenaltySample(rows, vocab, ids, reward, tokens, ws)}
    if kind == "ppl":
        b, n, vocab = case["batch"], case["n"], case["vocab"]
        logits = I.make_logits(0, 0, int(seed), device=dev, shape=(b, n, vocab))
        tokens = torch.from_numpy(I.make_answer_tokens(b, n, vocab, int(seed))).to(dev)
        # a confident model: the answer tokens hold most of their rows' probability
        logits.scatter_(2, tokens.long()[:, :, None], 3.0 * math.sqrt(2.0 * math.log(vocab)) + 4.0)
        return {"kind": kind, "logits": logits, "tokens": tokens,
                "ppl": torch.empty(b, dtype=torch.float32, device=dev),
                "stop": torch.empty(b, dtype=torch.int32, device=dev),
                "ws": torch.empty(B.answer_ppl_workspace_size(b, n, vocab), dtype=torch.uint8, device=dev)}
    # a decoder in the middle of its trajectory: the previous step's tokens are in the cache
    ci, qs, ks, vs, logits, ids = _loop_inputs(case, seed)
    dec = RecoDecoder(B.KVCache(ci.k, ci.v, ci.length), case["hq"], RecoPolicy(retention="clamp", window=case["w"]),
                      ci.q_win, ids)
    for q, kn, vn in zip(qs, ks, vs):
        dec.decode(q, kn, vn)
    return {"kind": kind, "dec": dec, "qs": qs, "ks": ks, "vs": vs, "logits": logits, "seed": int(seed),
            "rewards": [case["reward"]] * case["batch"]}


def run(s):
    kind = s["kind"]
    if kind == "decode":
        cache = s["cache"]
        if s["graph"] is not None:
            s["graph"].replay()
        else:
            s["call"](s["q"], s["kn"], s["vn"])
            if s["kn"] is not None:
                cache.length.sub_(1)                      # take the token back, so that every pass sees the same rows
        return {"out": s["out"], "lse": s["lse"], "k": cache.k, "v": cache.v}
    if kind == "score":
        c = s["case"]
        return B.reco_score(s["cache"], s["q"], c["w"], causal=c["causal"], scores=s["scores"], ws=s["ws"],
                            row_stats=s["stats"])
    if kind == "select":
        c, cache = s["case"], s["cache"]
        cache.length.copy_(s["full"])                     # every pass compresses the whole cache
        ranked = s["scores"]
        if s["pooled"] is not None:
            ranked = B.reco_pool_scores(cache, ranked, c["w"], c["pool"], "max", pooled=s["pooled"])
        B.reco_select_compact(cache, ranked, s["r"], c["w"], kept_idx=s["kept"], ws=s["ws"])
        return {"k": cache.k, "v": cache.v, "length": cache.length, "kept": s["kept"]}
    if kind == "sample":
        tokens = s["call"](s["logits"], *TAUS_BETAS, s["case"]["temperature"], s["seed"], 7)
        return {"logits": s["logits"], "tokens": tokens}
    if kind == "ppl":
        ppl, stop = B.reco_answer_ppl(s["logits"], s["tokens"], 1.1, ppl=s["ppl"], stop=s["stop"], ws=s["ws"])
        return {"ppl": ppl, "stop": stop}
    dec = s["dec"]
    dec.end_step(s["rewards"])
    for q, kn, vn, z in zip(s["qs"], s["ks"], s["vs"], s["logits"]):
        out, lse = dec.decode(q, kn, vn)
        tokens = dec.sample(z, 1.0, s["seed"])
    return {"out": out, "lse": lse, "scores": dec.scores, "length": dec.cache.length, "tokens": tokens,
            "logits": s["logits"]}


# ------------------------------------------------------------------ floors and tolerances
def _rows_total(case):
    return case["layers"] * case["hkv"] * int(_lens(case).sum())


def _kept(n, w, r):
    return min(n, max(min(w, n), math.ceil(r * n)))


def _decode_work(case, rows, layers):
    d, e = case["dim"], _elem(case)
    units, heads = layers * case["batch"] * case["hkv"], layers * case["batch"] * case["hq"]
    new = units if case.get("append", True) else 0
    return {"bytes": (rows + 2 * new) * 2 * d * e + heads * (2 * d * e + 4),
            "flops": 4.0 * d * (rows + new) * (case["hq"] // case["hkv"])}


def work(case):
    kind = case["kind"]
    if kind == "decode":
        return _decode_work(case, _rows_total(case), case["layers"])
    if kind == "score":
        rows, d, e, G, w = _rows_total(case), case["dim"], _elem(case), case["hq"] // case["hkv"], case["w"]
        heads = case["layers"] * case["batch"] * case["hq"]
        return {"bytes": rows * (d * e + 4) + heads * w * (d * e + (8 if case["fed"] else 0)),
                "flops": 2.0 * rows * G * w * d}
    if kind == "select":
        units, lens = case["layers"] * case["hkv"], _lens(case)
        kept = sum(_kept(int(n), case["w"], r)
                   for n, r in zip(lens, np.linspace(case["r_lo"], case["r_hi"], case["batch"])))
        moved = units * kept * 2 * case["dim"] * _elem(case)
        return {"bytes": units * int(lens.sum()) * 4 + units * kept * 4 + 2 * moved, "flops": 0}
    if kind == "sample":
        return {"bytes": case["rows"] * case["vocab"] * 4 + case["rows"] * case["ids"] * 4, "flops": 0}
    if kind == "ppl":
        return {"bytes": case["batch"] * case["n"] * case["vocab"] * 4, "flops": 0}
    # the loop: a scoring, a compaction, and the tokens' decode and sampling over the mean of the rows they see
    n, t = case["lo"] + case["tokens"], case["tokens"]
    units = case["layers"] * case["batch"] * case["hkv"]
    e, d = _elem(case), case["dim"]
    one = _decode_work(case, units * (case["lo"] + t // 2), case["layers"])
    byt = t * (one["bytes"] + case["batch"] * case["vocab"] * 4) + units * n * (d * e + 8) + 4 * units * case["lo"] * d * e
    return {"bytes": byt, "flops": t * one["flops"] + 2.0 * units * n * (case["hq"] // case["hkv"]) * case["w"] * d}


def tolerance(case):
    kind = case["kind"]
    if kind in ("select", "sample"):
        return "exact"                         # whole positions, moved rows, one fp32 subtraction per penalised logit
    if kind == "decode" or kind == "loop":
        # bf16: probabilities and results are rounded to 8 bits; fp32: sums in another order
        return {"rel": 1e-2, "max": 0.1} if case["dtype"] == "bf16" else {"rel": 4e-6, "max": 1e-4}
    if kind == "score":
        return {"rel": 4e-6, "max": 1e-4}      # fp32 sums and exponentials
    return {"rel": 1e-5, "max": 1e-4}          # the exponential of an fp32 log-likelihood


def _attend64(case, k, v, q):
    """fp64 attention of G queries [G][D] over rows k, v [n][D]: (out [G][D], lse [G])."""
    x = torch.matmul(q.double(), k.double().T.contiguous()) * _scale(case)
    lse = torch.logsumexp(x, -1)
    return torch.matmul(torch.exp(x - lse[:, None]), v.double()), lse


def exact(case, seed):
    kind = case["kind"]
    if kind in ("select", "sample"):
        return None
    if kind == "ppl":
        s = prepare_logits_only(case, seed)
        lse = torch.logsumexp(s[0].double(), -1)
        z = s[0].double().gather(2, s[1].long()[:, :, None])[:, :, 0]
        return {"ppl": torch.exp((lse - z).mean(-1)), "stop": None}
    G = case["hq"] // case["hkv"]
    if kind == "decode":
        ci, q, kn, vn = _decode_inputs(case, seed)
        out, lse = torch.zeros(q.shape, dtype=torch.float64, device=q.device), \
            torch.zeros(q.shape[:3], dtype=torch.float64, device=q.device)
        for l in range(case["layers"]):
            for b in range(case["batch"]):
                n = int(ci.seq_len[b])
                for h in range(case["hkv"]):
                    k, v = ci.k[l, b, h, :n], ci.v[l, b, h, :n]
                    if case["append"]:
                        k, v = torch.cat([k, kn[l, b, h][None]]), torch.cat([v, vn[l, b, h][None]])
                    o, z = _attend64(case, k, v, q[l, b, h * G:(h + 1) * G])
                    out[l, b, h * G:(h + 1) * G], lse[l, b, h * G:(h + 1) * G] = o, z
        return {"out": out, "lse": lse, "k": None, "v": None}
    if kind == "score":
        wl, ci = _cache(case, seed, case["hq"], case["w"], 64)
        return _scores64(case, ci)
    # the loop: the boundary's scores and selection, then the step's last token
    ci, qs, ks, vs, logits, ids = _loop_inputs(case, seed)
    n0, t, w = case["lo"], case["tokens"], case["w"]
    n = n0 + t
    ci.k[:, :, :, n0:n], ci.v[:, :, :, n0:n] = torch.stack(ks, 3), torch.stack(vs, 3)
    ci.q_win = torch.stack(qs[-w:], 3).contiguous()
    ci.seq_len = np.full(case["batch"], n)
    scores = _scores64(case, ci)
    m = _kept(n, w, 1.0 - 0.5 * case["reward"])
    out = torch.zeros(qs[0].shape, dtype=torch.float64, device=ci.k.device)
    lse = torch.zeros(qs[0].shape[:3], dtype=torch.float64, device=ci.k.device)
    for l in range(case["layers"]):
        for b in range(case["batch"]):
            for h in range(case["hkv"]):
                best = torch.sort(-scores[l, b, h, :n - w], stable=True).indices[:m - w]
                keep = torch.cat([best.sort().values, torch.arange(n - w, n, device=best.device)])
                k, v = (torch.cat([x[l, b, h][keep], torch.stack([y[l, b, h] for y in new])])
                        for x, new in ((ci.k, ks), (ci.v, vs)))
                o, z = _attend64(case, k, v, qs[-1][l, b, h * G:(h + 1) * G])
                out[l, b, h * G:(h + 1) * G], lse[l, b, h * G:(h + 1) * G] = o, z
    return {"out": out, "lse": lse, "scores": scores, "length": None, "tokens": None, "logits": None}


def prepare_logits_only(case, seed):
    s = prepare(case, seed)
    return s["logits"], s["tokens"]


def _scores64(case, ci):
    G = case["hq"] // case["hkv"]
    s = torch.zeros(ci.k.shape[:4], dtype=torch.float64, device=ci.k.device)
    for l in range(case["layers"]):
        for b in range(case["batch"]):
            n = int(ci.seq_len[b])
            for h in range(case["hkv"]):
                x = _logits64(case, ci.k[l, b, h, :n], ci.q_win[l, b, h * G:(h + 1) * G], case.get("causal", True))
                s[l, b, h, :n] = torch.softmax(x, -1).sum((0, 1))
    return s
