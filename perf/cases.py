"""The calls this framework is timed on: decode steps, prompt processing and the weight update of rollout generation,
each through the library's public entry points (paper_2511_00796_amd.binding), over the range of sizes it is used at.

A case is one of three operations:

  decode   one decode_step / decode_step_sample / decode_step_top_p of `batch` sequences whose caches hold `lo`..`hi`
           tokens (`law` uniform or loguniform), in a bf16 or 8-bit cache.
  prefill  `tokens` prompt tokens of `prompts` prompts that each have `cached` tokens in the cache already: whole blocks
           of 256 rows through prefill_rows, the rest through prefill_chunk.  out "kv": all prompt tokens go in and the
           cache is read back (a prefill worker that hands the cache on); out "first_token": the last token of every
           prompt goes through decode_step, as when a rollout starts.
  update   new weights are packed into a live engine (every layer and the globals), then one decode step runs.

Model shapes are the repository's own (synth.py); `layers` truncates the depth, so that a case is a few layers of the
model -- every layer of a model does the same work -- and a rounding difference is not carried through 28 of them.  Two
cases are whole models.  Sampled tokens are not among the outputs (two rounding-equal evaluations may draw another token
at a near tie, and one token is more than a hundredth of most batches); logits and log-probabilities are.
"""
import dataclasses
import math

import numpy as np
import torch

from paper_2511_00796_amd import binding, synth

SHAPES = {"tiny": synth.TINY, "1.5b": synth.QWEN_1P5B, "7b": synth.QWEN_7B, "14b": synth.QWEN_14B}
DEV = "cuda:0"
SPARE_BLOCKS = 8


def _decode(name, model, layers, batch, lo, hi, law="uniform", kv="bf16", head="greedy", op="decode"):
    c = {"op": op, "model": model, "layers": layers, "batch": batch, "lo": lo, "hi": hi, "law": law, "kv": kv, "head": head}
    return dict(c, name=name) if name else c


def _prefill(name, model, layers, tokens, prompts, cached=0, kv="bf16", out="kv"):
    c = {"op": "prefill", "model": model, "layers": layers, "tokens": tokens, "prompts": prompts, "cached": cached, "kv": kv,
         "out": out}
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: a whole two-layer model, four short sequences; launches and latency are all there is
        _decode("decode-tiny-b4", "tiny", 2, 4, 32, 128),
        # a whole 1.5B model in the middle of a rollout, all 28 layers
        _decode("decode-1.5b-b64-whole", "1.5b", 28, 64, 512, 8192),
        # the headline configuration: 7B, 128 long ragged sequences, tokens drawn at temperature 1 as rollouts are
        _decode("decode-7b-b128", "7b", 4, 128, 1024, 16384, head="sample"),
        # the same batch over the 8-bit cache
        _decode("decode-7b-b128-fp8", "7b", 4, 128, 1024, 16384, kv="fp8", head="sample"),
        # the largest model, nucleus sampling
        _decode("decode-14b-b64-top-p", "14b", 4, 64, 1024, 16384, head="top_p"),
        # the largest batch with skewed lengths, as rollout lengths are
        _decode("decode-1.5b-b256-longtail", "1.5b", 4, 256, 256, 16384, law="loguniform", head="sample"),
        # the end of a rollout: three very long responses are left
        _decode("decode-7b-b3-tail", "7b", 4, 3, 8192, 32768, head="sample"),
        # the beginning of one, an odd number of short, very uneven sequences
        _decode("decode-7b-b37-short", "7b", 4, 37, 1, 3000, head="sample"),
        # the last, odd piece of a prompt whose beginning is in the cache already, up to its first generated token
        _prefill("prompt-1.5b-201-cached", "1.5b", 4, 201, 1, cached=3000, out="first_token"),
        # one ordinary prompt
        _prefill("prompt-7b-2048", "7b", 4, 2048, 1),
        # seven uneven prompts of an odd total, largest model, 8-bit cache, up to their first tokens
        _prefill("prompt-14b-5000-fp8", "14b", 3, 5000, 7, kv="fp8", out="first_token"),
        # the policy update: new weights into the live engine, then a step
        _decode("update-7b-b16", "7b", 4, 16, 256, 4096, head="sample", op="update"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


KV_CAP = 9.0e9          # bytes of cache a drawn decode case may read: about the listed ones'


def draw(rng):
    model = rng.choice(["tiny", "1.5b", "7b", "7b", "14b"])
    layers = 2 if model == "tiny" else rng.randint(2, 4)
    kind = rng.choice(["decode"] * 6 + ["prefill"] * 3 + ["update"])
    kv = rng.choice(["bf16", "bf16", "fp8"])
    if kind == "prefill":
        out = rng.choice(["kv", "first_token"])
        tokens = _log(rng, 20, 5000)
        prompts = min(_log(rng, 1, 24), max(1, tokens // 8))
        cached = rng.choice([0, 0, _log(rng, 16, 6000)]) if out == "first_token" else 0
        cached = cached if prompts <= 4 else min(cached, 1000)
        return _prefill(None, model, min(layers, 3), tokens, prompts, cached, kv if out == "first_token" else "bf16", out)
    batch = _log(rng, 1, 256)
    hi = _log(rng, 64, 32768)
    per_token = SHAPES[model].kv_bytes_per_token() / SHAPES[model].n_layers * layers * (0.5 if kv == "fp8" else 1.0)
    hi = max(64, min(hi, int(KV_CAP / per_token / batch)))
    lo = max(1, int(hi * rng.uniform(0.02, 0.9)))
    return _decode(None, model, layers, batch, lo, hi, rng.choice(["uniform", "loguniform"]), kv,
                   rng.choice(["greedy", "sample", "top_p"]), kind)


# ---- inputs ---------------------------------------------------------------------------------------------------------
TEMPERATURE, TOP_P, SAMPLE_SEED = 0.9, 0.95, 77


def _shape(case):
    return dataclasses.replace(SHAPES[case["model"]], n_layers=case["layers"])


def _lengths(case):
    """Tokens cached per sequence (decode) or prompt tokens per prompt (prefill): a property of the case, not of the seed."""
    if case["op"] == "prefill":
        n, p = case["tokens"], case["prompts"]
        r = np.random.default_rng(n * 31 + p)
        share = r.uniform(0.2, 1.0, p)
        lens = np.maximum(2, np.floor(share / share.sum() * n).astype(np.int64))
        lens[0] += n - lens.sum()
        return lens.astype(np.int32)
    b, lo, hi = case["batch"], case["lo"], case["hi"]
    r = np.random.default_rng(b * 1000003 + lo * 1009 + hi)
    if case["law"] == "loguniform":
        v = np.rint(np.exp(r.uniform(math.log(lo), math.log(hi), b)))
    else:
        v = r.integers(lo, hi + 1, b)
    return np.clip(v, lo, hi).astype(np.int32)


def _gen(seed, kind, layer=0):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + kind * 10007 + layer * 101 + 17) % (2 ** 62))
    return g


def _normal(shape, std, g, mean=0.0):
    t = torch.randn(shape, generator=g, device=DEV, dtype=torch.bfloat16)
    if std != 1.0:
        t.mul_(std)
    return t.add_(mean) if mean else t


def _layer(s, l, seed):
    """One layer's weights, logical [in, out] bf16; gate and up as a trained model's would be, N(0, 0.02^2)."""
    g = _gen(seed, 1, l)
    return {"g1": _normal((s.hidden,), 0.02, g, 1.0), "wqkv": _normal((s.hidden, s.qkv_dim), 0.02, g),
            "bqkv": _normal((s.qkv_dim,), 0.02, g), "wo": _normal((s.q_dim, s.hidden), 0.02, g),
            "g2": _normal((s.hidden,), 0.02, g, 1.0), "wg": _normal((s.hidden, s.intermediate), 0.02, g),
            "wu": _normal((s.hidden, s.intermediate), 0.02, g), "wd": _normal((s.intermediate, s.hidden), 0.02, g)}


def _globals(s, seed):
    g = _gen(seed, 2)
    return {"embed": _normal((s.vocab, s.hidden), 0.02, g), "gf": _normal((s.hidden,), 0.02, g, 1.0),
            "wlm": _normal((s.hidden, s.vocab), 0.02, g)}


def _kv_fill(s, l, total, seed):
    g = _gen(seed, 3, l)
    return _normal((total, s.n_kv_heads, s.head_dim), 1.0, g), _normal((total, s.n_kv_heads, s.head_dim), 1.0, g)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _tokens(case, seed):
    s = _shape(case)
    n = case["tokens"] if case["op"] == "prefill" else case["batch"]
    return np.random.default_rng(int(seed) + 5).integers(0, s.vocab, n).astype(np.int32)


def _table(need, seed, extra=SPARE_BLOCKS):
    ids = np.random.default_rng(int(seed) + 9).permutation(int(need.sum()) + extra).astype(np.int32)
    table = np.zeros((len(need), int(need.max())), np.int32)
    at = 0
    for b, n in enumerate(need):
        table[b, :n] = ids[at:at + n]
        at += int(n)
    return table, len(ids)


def _starts(lens):
    return np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)


def prepare(case, seed):
    s = _shape(case)
    prefill = case["op"] == "prefill"
    lens = _lengths(case)
    cached = np.full(len(lens), case["cached"], np.int32) if prefill else lens      # tokens in the cache before the call
    after = cached + lens if prefill else lens + 1
    kvt = binding.HX_KV_FP8_E4M3 if case["kv"] == "fp8" else binding.HX_KV_BF16
    eng = binding.Engine(s, 256 if prefill else case["batch"], int(after.max()), device=DEV, kv_dtype=kvt)
    table, blocks = _table((after + 15) // 16, seed)
    kv = binding.KVCache(eng, blocks)
    table_d, start_d = _dev(table), _dev(_starts(cached))
    st = {"case": case, "eng": eng, "kv": kv, "table": table_d}
    weights = []
    for l in range(s.n_layers):
        w = _layer(s, l, seed)
        eng.pack_layer(l, _layer(s, l, seed + 1) if case["op"] == "update" else w)
        if case["op"] == "update":
            weights.append(w)
        if int(cached.sum()):
            k, v = _kv_fill(s, l, int(cached.sum()), seed)
            kv.prefill_fill(l, k, v, start_d, table_d)
            del k, v
        del w
    g = _globals(s, seed)
    eng.pack_globals(_globals(s, seed + 1) if case["op"] == "update" else g)
    toks = _tokens(case, seed)
    if prefill:
        starts = _starts(lens)
        seq = np.repeat(np.arange(len(lens)), lens)
        pos = np.arange(len(seq), dtype=np.int64) - starts[seq] + cached[seq]
        rows = np.ones(len(seq), bool)
        if case["out"] == "first_token":
            rows[starts[1:] - 1] = False
            last = starts[1:] - 1
            st["last"] = tuple(_dev(x.astype(np.int32)) for x in (toks[last], pos[last], pos[last] + 1))
            st["logits"] = torch.empty(len(lens), s.vocab, dtype=torch.float32, device=DEV)
            st["next"] = torch.empty(len(lens), dtype=torch.int32, device=DEV)
        r = np.nonzero(rows)[0]
        wide = len(r) // 256 * 256

        def args(ix):
            return tuple(_dev(x.astype(np.int32)) for x in (toks[ix], pos[ix], pos[ix] + 1, table[seq[ix]]))
        st["wide"] = args(r[:wide]) if wide else None
        st["rest"] = args(r[wide:]) if len(r) > wide else None
        st["ws"] = torch.empty(binding.prefill_workspace_bytes(eng.cfg, wide), dtype=torch.uint8, device=DEV) if wide else None
        st["starts"], st["total"] = _dev(starts), int(lens.sum())
    else:
        st["step"] = tuple(_dev(x.astype(np.int32)) for x in (toks, lens, lens + 1))
        st["logits"] = torch.empty(case["batch"], s.vocab, dtype=torch.float32, device=DEV)
        st["next"] = torch.empty(case["batch"], dtype=torch.int32, device=DEV)
        st["logprobs"] = torch.empty(case["batch"], dtype=torch.float32, device=DEV)
        if case["op"] == "update":
            st["weights"], st["globals"] = weights, g
    return st


def run(st):
    case, eng, kv, table = st["case"], st["eng"], st["kv"], st["table"]
    if case["op"] == "prefill":
        if st["wide"] is not None:
            eng.prefill_rows(kv, *st["wide"], st["ws"])
        if st["rest"] is not None:
            eng.prefill_chunk(kv, *st["rest"])
        if case["out"] == "first_token":
            tok, pos, lens = st["last"]
            eng.decode_step(kv, tok, pos, lens, table, st["logits"], st["next"])
            return {"logits": st["logits"]}
        return [kv.gather(l, st["total"], st["starts"], table) for l in range(case["layers"])]
    if case["op"] == "update":
        for l, w in enumerate(st["weights"]):
            eng.pack_layer(l, w)
        eng.pack_globals(st["globals"])
    tok, pos, lens = st["step"]
    if case["head"] == "greedy":
        eng.decode_step(kv, tok, pos, lens, table, st["logits"], st["next"])
        return {"logits": st["logits"]}
    if case["head"] == "sample":
        eng.decode_step_sample(kv, tok, pos, lens, table, TEMPERATURE, SAMPLE_SEED, st["logits"], st["next"], st["logprobs"])
    else:
        eng.decode_step_top_p(kv, tok, pos, lens, table, TEMPERATURE, TOP_P, SAMPLE_SEED, st["logits"], st["next"],
                              st["logprobs"])
    return {"logits": st["logits"], "logprobs": st["logprobs"]}


# ---- what a pass cannot do without ----------------------------------------------------------------------------------
def work(case):
    s = _shape(case)
    lens = _lengths(case).astype(np.int64)
    elem = 1 if case["kv"] == "fp8" else 2
    kv_token = 2 * s.kv_dim * elem                                      # per layer
    per_layer = s.hidden * s.qkv_dim + s.q_dim * s.hidden + 3 * s.hidden * s.intermediate
    vec = s.qkv_dim + 2 * s.hidden
    head = s.hidden * s.vocab
    L = s.n_layers

    def step(b, keys):                                                  # a decode step: weights, K and V once, logits out
        return (2 * (L * (per_layer + vec) + head + s.hidden) + L * kv_token * (keys + b) + 2 * b * s.hidden + 4 * b * s.vocab,
                2 * b * (L * per_layer + head) + L * 4 * keys * s.q_dim)
    if case["op"] != "prefill":
        by, fl = step(case["batch"], int((lens + 1).sum()))
        if case["op"] == "update":
            by += 2 * 2 * (L * (per_layer + vec) + head + s.hidden * s.vocab + s.hidden)
        return {"bytes": by, "flops": fl}
    first = case["out"] == "first_token"
    n = lens - 1 if first else lens
    rows = int(n.sum())
    attended = int((n * case["cached"] + n * (n + 1) // 2).sum())
    by = 2 * ((L - 1) * per_layer + s.hidden * s.qkv_dim) + 2 * rows * s.hidden + L * kv_token * rows
    by += (L - 1) * kv_token * case["cached"] * len(lens)
    fl = 2 * rows * ((L - 1) * per_layer + s.hidden * s.qkv_dim) + (L - 1) * 4 * attended * s.q_dim
    if first:
        b2, f2 = step(len(lens), int((lens + case["cached"]).sum()))
        by, fl = by + b2, fl + f2
    else:
        by += 2 * L * 2 * s.kv_dim * int(lens.sum()) * 2                 # the cache read back: read and written once
    return {"bytes": by, "flops": fl}


def tolerance(case):
    """Measured by the same inputs under other orders of summation (other K-splits, other cuts of the attention, rows
    attended one by one): a rounding flip of a bf16 activation travels through the layers that follow.  One layer and the
    head: 0.0016 to 0.0027; two: 0.0036 to 0.0053; three: 0.0045 to 0.0076; four: 0.0039 to 0.010 (the larger ones with
    an 8-bit cache, or where a drawn token at a near tie took its log-probability along); 28: 0.015.  Largest single
    difference: 0.13 of the root mean square."""
    return {"rel": min(0.03, 0.01 + 0.005 * case["layers"]), "max": 0.5}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------
def exact(case, seed):
    """Plain torch in float64, nothing rounded on the way but what an 8-bit cache stores."""
    s = _shape(case)
    prefill = case["op"] == "prefill"
    lens = _lengths(case)
    cached = np.full(len(lens), case["cached"], np.int32) if prefill else lens
    new = lens if prefill else np.ones_like(lens)                       # rows per sequence
    starts, cstarts = _starts(new), _starts(cached)
    seq = np.repeat(np.arange(len(new)), new)
    pos = torch.from_numpy(np.arange(len(seq)) - starts[seq] + cached[seq]).to(DEV, torch.float64)
    G, D, nq, nk = s.group, s.head_dim, s.n_q_heads, s.n_kv_heads
    ang = pos[:, None] * (float(s.rope_theta) ** (-torch.arange(D // 2, device=DEV, dtype=torch.float64) / (D // 2)))[None]
    cos, sin = ang.cos()[:, None], ang.sin()[:, None]

    def norm(x, gain):
        return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * gain.double()

    def rope(t):
        a, b = t[..., :D // 2], t[..., D // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)

    def stored(t):
        return t.float().to(torch.float8_e4m3fn).double() if case["kv"] == "fp8" else t

    g = _globals(s, seed)
    x = g["embed"][_dev(_tokens(case, seed)).long()].double()
    kv_out = []
    for l in range(s.n_layers):
        w = _layer(s, l, seed)
        qkv = norm(x, w["g1"]) @ w["wqkv"].double() + w["bqkv"].double()
        q = rope(qkv[:, :nq * D].reshape(-1, nq, D))
        k = stored(rope(qkv[:, nq * D:(nq + nk) * D].reshape(-1, nk, D)))
        v = stored(qkv[:, (nq + nk) * D:].reshape(-1, nk, D))
        if prefill and case["out"] == "kv":
            kv_out.append((k, v))
            if l + 1 == s.n_layers:
                return kv_out
        ck, cv = _kv_fill(s, l, int(cached.sum()), seed) if int(cached.sum()) else (None, None)
        o = torch.empty(len(seq), nq, D, device=DEV, dtype=torch.float64)
        for b in range(len(new)):
            r0, r1, n, c = int(starts[b]), int(starts[b + 1]), int(new[b]), int(cached[b])
            kb, vb = k[r0:r1], v[r0:r1]
            if c:
                kb = torch.cat([stored(ck[cstarts[b]:cstarts[b + 1]].double()), kb])
                vb = torch.cat([stored(cv[cstarts[b]:cstarts[b + 1]].double()), vb])
            mask = None
            if n > 1:
                mask = torch.arange(c + n, device=DEV)[None] > torch.arange(c, c + n, device=DEV)[:, None]
            for h in range(nk):
                kh, vh = kb[:, h].t().contiguous(), vb[:, h].contiguous()
                if n == 1:
                    o[r0, h * G:(h + 1) * G] = torch.softmax(q[r0, h * G:(h + 1) * G] @ kh / math.sqrt(D), -1) @ vh
                    continue
                for j in range(h * G, (h + 1) * G):
                    sc = (q[r0:r1, j] @ kh / math.sqrt(D)).masked_fill_(mask, -math.inf)
                    o[r0:r1, j] = torch.softmax(sc, -1) @ vh
        del ck, cv
        x = x + o.reshape(len(seq), -1) @ w["wo"].double()
        u = norm(x, w["g2"])
        gate = u @ w["wg"].double()
        x = x + (gate * torch.sigmoid(gate) * (u @ w["wu"].double())) @ w["wd"].double()
    if prefill:
        x = x[torch.from_numpy(starts[1:] - 1).to(DEV).long()]
    logits = norm(x, g["gf"]) @ g["wlm"].double()
    if prefill or case["head"] == "greedy":
        return {"logits": logits}
    return {"logits": logits, "logprobs": None}                        # which token is drawn hangs on the generator
