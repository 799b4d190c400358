"""What the speed of this library is measured on: the calls that a program with an SP-KV cache
makes, each through the public binding, over the range of sizes it is used at.

A case describes one attention layer (heads, head_dim, window, tau), the prompts its cache holds
(batch, ctx_min .. ctx_max tokens, gated on at keep_min .. keep_max per KV head) and the call:

  step      decode_step: append and decode of one new token per sequence
  predict   decode_step_predict: the same with the utility predictor inside
  attend    append, then decode_attention: the step as two calls
  score     score_chunk of `tokens` drafts per sequence, then append of the accepted ones
  chunk     decode_chunk of `tokens` new tokens per sequence
  prefill   reset, then prefill_attention over whole prompts in pieces of `tokens` tokens
  feed      reset, then append of whole prompts in such pieces, then the first decode_attention
  soft      soft_gated_attention over whole packed sequences (the training-time forward)
  logits    utility_logits of `tokens` hidden states

The decoding kinds are run thousands of times on one state.  The tokens they bring therefore
nearly all fail the gate (one in 256 passes): lists stay as long as the prompts left them.
"""

from __future__ import annotations

import math

import torch

import paper_2605_14037_amd as spkv

PASSES = 65536          # passes that a decoding state has room for
GEN_KEEP = 1.0 / 256    # keep rate of the tokens that the decoding kinds bring
RING = 16               # different sets of new tokens, used in turn


def _case(name, kind, **kw):
    c = {"name": name, "kind": kind, "batch": 1, "q_heads": 32, "kv_heads": 8, "head_dim": 128,
         "ctx_min": 0, "ctx_max": 0, "keep_min": 0.10, "keep_max": 0.33, "mixed": False,
         "window": 128, "tau": 0.5, "tokens": 1, "d_model": 0, "d_hidden": 0}
    c.update(kw)
    return c


def listed():
    return [
        # one short conversation on a small model: launches and host work
        _case("step_b1_2k_d64", "step", q_heads=8, kv_heads=2, head_dim=64, ctx_min=2048, ctx_max=2048),
        # the usual serving step: an 8B-shaped layer, 16 sequences of 32k tokens
        _case("step_b16_32k", "step", batch=16, ctx_min=32768, ctx_max=32768),
        # long documents, few sequences
        _case("step_b4_128k", "step", batch=4, ctx_min=131072, ctx_max=131072, keep_min=0.02,
              keep_max=0.15),
        # a full server: 64 requests of all ages, dense, local and sparse heads (the largest cache)
        _case("step_b64_ragged_mixed", "step", batch=64, ctx_min=1024, ctx_max=65536, keep_min=0.05,
              keep_max=0.30, mixed=True),
        # one layer of a model that computes its own gates: predictor inside the step
        _case("predict_b32_16k", "predict", batch=32, ctx_min=16384, ctx_max=16384, keep_min=0.15,
              keep_max=0.15, d_model=4096, d_hidden=256),
        # a runtime that appends and attends separately; odd sizes, small heads, ragged prompts
        _case("attend_b7_odd_d64", "attend", batch=7, q_heads=24, kv_heads=3, head_dim=64,
              ctx_min=901, ctx_max=9973, window=100, tau=0.3),
        # speculative decoding: four drafts scored, the accepted ones appended
        _case("score4_b16_32k", "score", batch=16, ctx_min=32768, ctx_max=32768, tokens=4),
        # 16-token chunks per sequence (chunked prompts beside decoding)
        _case("chunk16_b16_32k", "chunk", batch=16, ctx_min=32768, ctx_max=32768, tokens=16),
        # prompts with their own attention, ragged lengths, pieces of 4096 tokens
        _case("prefill_b4_ragged_16k", "prefill", batch=4, ctx_min=3001, ctx_max=19531, tokens=4096),
        # prompts whose attention is computed elsewhere: the write path alone
        _case("feed_b16_32k", "feed", batch=16, ctx_min=32768, ctx_max=32768, tokens=4096),
        # training-time forward, whole sequences (the most arithmetic)
        _case("soft_b4_16k", "soft", batch=4, ctx_min=16001, ctx_max=16384),
        # gate logits of a prompt piece
        _case("logits_32k", "logits", tokens=32768, d_model=4096, d_hidden=256),
    ]


SHAPES = [(32, 8, 128), (32, 8, 128), (8, 2, 64), (16, 2, 128), (24, 3, 64), (16, 1, 128), (8, 8, 128)]


def draw(rng):
    """One more case: sizes over the whole range of the listed ones, odd ones among them."""
    def span(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["step", "step", "step", "predict", "attend", "score", "chunk", "prefill",
                       "feed", "soft", "logits"])
    hq, hk, d = rng.choice(SHAPES)
    c = _case("", kind, q_heads=hq, kv_heads=hk, head_dim=d, tau=rng.choice([0.5, 0.5, 0.3, 0.7]),
              window=rng.choice([128, 128, 64, span(16, 512)]))
    del c["name"]
    c["keep_min"] = round(rng.uniform(0.02, 0.15), 3)
    c["keep_max"] = round(c["keep_min"] + rng.uniform(0.0, 0.25), 3)
    if kind == "logits":
        c.update(tokens=span(1, 32768), d_model=128 * rng.randint(4, 32),
                 d_hidden=16 * rng.choice([4, 8, 16, rng.randint(2, 16)]))
        return c
    if kind == "soft":
        c["batch"] = rng.randint(1, 4)
        c["ctx_max"] = span(256, 16000)
    elif kind in ("prefill", "feed"):
        c["batch"] = rng.randint(1, 4 if kind == "prefill" else 16)
        c["ctx_max"] = span(512, 19531 if kind == "prefill" else 32768)
        c["tokens"] = rng.choice([4096, 2048, span(100, 4096)])
        c["tokens"] = max(c["tokens"], -(-c["ctx_max"] // 16))       # at most 16 pieces
    else:
        c["batch"] = span(1, 64)
        c["ctx_max"] = span(512, min(131072, 1048576 // c["batch"]))
        c["mixed"] = rng.random() < 0.2
        if kind in ("score", "chunk"):
            most = min(16, c["window"], 64 // (hq // hk))
            c["tokens"] = rng.randint(2, most)
        if kind == "predict":
            c.update(d_model=128 * rng.randint(4, 32), d_hidden=16 * rng.randint(2, 16))
    c["ctx_min"] = c["ctx_max"] if rng.random() < 0.4 else max(1, int(c["ctx_max"] * rng.uniform(0.05, 1.0)))
    return c


# ------------------------------------------------------------------------------- inputs
def _frac(i):
    return (0.6180339887498949 * (i + 1)) % 1.0


def _lens(c):
    return [c["ctx_min"] + int(_frac(b) * (c["ctx_max"] - c["ctx_min"] + 1)) for b in range(c["batch"])]


def _keep(c):
    """Keep rate of every (sequence, KV head): by head, or a quarter dense, a quarter local-only."""
    rows = []
    for b in range(c["batch"]):
        row = []
        for h in range(c["kv_heads"]):
            i = b * c["kv_heads"] + h if c["mixed"] else h
            rate = c["keep_min"] + _frac(i) * (c["keep_max"] - c["keep_min"])
            kind = (5 * b + 3 * h) % 4 if c["mixed"] else 2
            row.append(1.0 if kind == 0 else 0.0 if kind == 1 else rate)
        rows.append(row)
    return torch.tensor(rows, dtype=torch.float64)


def _theta(c):
    tau = float(torch.tensor(c["tau"], dtype=torch.float32))
    return float(torch.tensor(math.log(tau / (1.0 - tau)), dtype=torch.float32))


def _mu(c, keep):
    mu = torch.special.ndtri(keep.clamp(1e-12, 1 - 1e-12))
    mu = torch.where(keep >= 1, 40.0, torch.where(keep <= 0, -40.0, mu))
    return (mu + _theta(c)).to(torch.float32).cuda()


def _gen(seed, part):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 8 + part)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32)


def _rows(c, g, counts, mu):
    """k, v, logits and cu_seqlens of counts[b] new tokens of every sequence b."""
    cu = [0]
    for n in counts:
        cu.append(cu[-1] + n)
    k = _randn(g, cu[-1], c["kv_heads"], c["head_dim"]).to(torch.bfloat16)
    v = _randn(g, cu[-1], c["kv_heads"], c["head_dim"]).to(torch.bfloat16)
    seq = torch.repeat_interleave(torch.arange(len(counts)), torch.tensor(counts)).cuda()
    return k, v, (_randn(g, cu[-1], c["kv_heads"]) + mu[seq]).contiguous(), cu


def _query(c, g, rows):
    return _randn(g, rows, c["q_heads"], c["head_dim"]).to(torch.bfloat16)


def _pieces(c, size):
    """Token counts that bring every sequence to its length, at most `size` tokens at a time."""
    lens, done = _lens(c), 0
    while done < max(lens):
        yield [max(0, min(size, n - done)) for n in lens]
        done += size


def _prompt(c, seed, size):
    g, mu = _gen(seed, 0), _mu(c, _keep(c))
    for counts in _pieces(c, size):
        yield _rows(c, g, counts, mu)


def _accepted(c):
    return [(3 * b + 1) % (c["tokens"] + 1) for b in range(c["batch"])]


def _new_tokens(c, seed):
    """RING sets of new tokens: (k, v, logits, cu, q) of `tokens` rows per sequence."""
    g = _gen(seed, 1)
    mu = _mu(c, torch.full((c["batch"], c["kv_heads"]), GEN_KEEP, dtype=torch.float64))
    got = []
    for _ in range(RING):
        k, v, f, cu = _rows(c, g, [c["tokens"]] * c["batch"], mu)
        got.append((k, v, f, cu, _query(c, g, cu[-1])))
    return got


def _predictor(c, seed, rows):
    """Hidden states and the two-layer predictor; its logits spread by about one around b2."""
    g, dm, dh, hk = _gen(seed, 2), c["d_model"], c["d_hidden"], c["kv_heads"]
    hidden = _randn(g, rows, dm).to(torch.bfloat16)
    w1 = (_randn(g, dh, dm) / math.sqrt(dm)).to(torch.bfloat16)
    b1 = _randn(g, dh) * 0.1
    w2 = (_randn(g, hk, dh) / (0.6 * math.sqrt(dh))).to(torch.bfloat16)
    b2 = _randn(g, hk) * 0.1 + (_theta(c) - 3.0)
    return hidden, w1, b1, w2, b2


def _cache(c, piece):
    pairs, lens = c["batch"] * c["kv_heads"], torch.tensor(_lens(c), dtype=torch.float64)
    kept = float((_keep(c) * lens[:, None]).sum())
    return spkv.SPKVCache(c["batch"], c["q_heads"], c["kv_heads"], c["head_dim"],
                          max_context=max(_lens(c)) + PASSES * min(c["tokens"], 16),
                          max_total_kept_tokens=int(1.08 * kept) + pairs * (min(piece, max(_lens(c))) + 512),
                          window=c["window"], tau=c["tau"])


def prepare(case, seed):
    c = dict(case)
    s = {"case": c, "kind": c["kind"], "at": 0}
    hq, d, hk = c["q_heads"], c["head_dim"], c["kv_heads"]

    def buffers(rows):
        return (torch.empty(rows, hq, d, dtype=torch.bfloat16, device="cuda"),
                torch.empty(rows, hq, dtype=torch.float32, device="cuda"))

    if c["kind"] == "logits":
        s["in"] = _predictor(c, seed, c["tokens"])
        s["out"] = torch.empty(c["tokens"], hk, dtype=torch.float32, device="cuda")
        s["ws"] = torch.empty(c["tokens"] * c["d_hidden"], dtype=torch.float32, device="cuda")
        return s
    if c["kind"] == "soft":
        k, v, f, cu = next(_prompt(c, seed, c["ctx_max"] + 1))
        s["in"] = (_query(c, _gen(seed, 3), cu[-1]), k, v, f, cu)
        s["out"] = torch.empty(cu[-1], hq, d, dtype=torch.bfloat16, device="cuda")
        need = spkv.load_library().spkv_soft_gated_workspace_bytes(c["batch"], hk, d, c["window"], max(_lens(c)))
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        return s
    if c["kind"] in ("prefill", "feed"):
        s["cache"] = cache = _cache(c, c["tokens"])
        g, s["in"] = _gen(seed, 3), []
        for k, v, f, cu in _prompt(c, seed, c["tokens"]):
            q, out, lse = None, None, None
            if c["kind"] == "prefill":
                q, (out, lse) = _query(c, g, cu[-1]), buffers(cu[-1])
            s["in"].append((k, v, f, q, cache.make_cu(cu), out, lse))
        if c["kind"] == "prefill":
            n_max = min(c["tokens"], max(_lens(c)))
            s["ws"] = torch.empty(cache.prefill_workspace_bytes(n_max, n_max * c["batch"]),
                                  dtype=torch.uint8, device="cuda")
        else:
            s["q"], (s["out"], s["lse"]) = _query(c, g, c["batch"]), buffers(c["batch"])
        return s
    s["cache"] = cache = _cache(c, 4096)
    for k, v, f, cu in _prompt(c, seed, 4096):
        cache.append(k, v, f, cu)
    s["in"] = [(k, v, f, cache.make_cu(cu), q) for k, v, f, cu, q in _new_tokens(c, seed)]
    s["out"], s["lse"] = buffers(c["batch"] * c["tokens"])
    if c["kind"] == "predict":
        s["net"] = _predictor(c, seed, c["batch"])
        s["logits"] = torch.empty(c["batch"], hk, dtype=torch.float32, device="cuda")
        need = cache.lib.spkv_decode_step_predict_workspace_bytes(c["batch"], c["d_hidden"])
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    if c["kind"] == "score":
        counts = _accepted(c)
        rows = torch.tensor([b * c["tokens"] + i for b, n in enumerate(counts) for i in range(n)],
                            dtype=torch.int64, device="cuda")
        s["acc"] = [tuple(x.index_select(0, rows) for x in t[:3]) for t in s["in"]]
        cu = [0]
        for n in counts:
            cu.append(cu[-1] + n)
        s["acc_cu"] = cache.make_cu(cu)
    return s


# ---------------------------------------------------------------------------------- run
def run(s):
    kind = s["kind"]
    if kind == "logits":
        return spkv.utility_logits(*s["in"], out=s["out"], workspace=s["ws"])
    if kind == "soft":
        return spkv.soft_gated_attention(*s["in"], window=s["case"]["window"], out=s["out"],
                                         want_lse=True, workspace=s["ws"])
    cache = s["cache"]
    if kind == "prefill":
        cache.reset()
        return [cache.prefill_attention(k, v, f, q, cu, workspace=s["ws"], out=out, lse=lse)
                for k, v, f, q, cu, out, lse in s["in"]]
    if kind == "feed":
        cache.reset()
        for k, v, f, _, cu, _, _ in s["in"]:
            cache.append(k, v, f, cu)
        return cache.decode_attention(s["q"], out=s["out"], lse=s["lse"])
    at = s["at"] % RING
    s["at"] += 1
    k, v, f, cu, q = s["in"][at]
    if kind == "step":
        return cache.decode_step(k, v, f, q, out=s["out"], lse=s["lse"])
    if kind == "predict":
        return cache.decode_step_predict(*s["net"], k, v, q, out=s["out"], lse=s["lse"],
                                         util_logits=s["logits"], workspace=s["ws"])
    if kind == "attend":
        cache.append(k, v, f, cu)
        return cache.decode_attention(q, out=s["out"], lse=s["lse"])
    if kind == "chunk":
        return cache.decode_chunk(k, v, f, q, cu, out=s["out"], lse=s["lse"])
    r = cache.score_chunk(k, v, q, cu, out=s["out"], lse=s["lse"])
    cache.append(*s["acc"][at], s["acc_cu"])
    return r


# --------------------------------------------------------------------- cost and accuracy
def _attended(c):
    """Sum over (KV head, query) of the keys that a query attends to, as expected from the keep
    rates, and the pairs the cache holds at the end."""
    keep, lens, w, n = _keep(c), _lens(c), c["window"], c["tokens"]
    keys = held = 0.0
    for b, t in enumerate(lens):
        rate = float(keep[b].sum())
        held += c["kv_heads"] * min(t, w) + rate * max(0, t - w)
        if c["kind"] in ("prefill", "feed"):
            far = max(0, t - w)
            keys += c["kv_heads"] * (t * min(t, w) - min(t, w) * (min(t, w) - 1) / 2.0) + rate * far * (far + 1) / 2.0
        elif c["kind"] == "soft":
            keys += c["kv_heads"] * t * (t + 1) / 2.0
        else:
            keys += n * (c["kv_heads"] * min(t + 1, w) + rate * max(0, t + 1 - w))
    return keys, held


def work(case):
    c = dict(case)
    dm, dh, hk, hq, d = c["d_model"], c["d_hidden"], c["kv_heads"], c["q_heads"], c["head_dim"]
    net_bytes = 2 * dm * dh + 4 * dh + 2 * hk * dh + 4 * hk
    if c["kind"] == "logits":
        n = c["tokens"]
        return {"bytes": 2 * n * dm + net_bytes + 4 * n * hk, "flops": 2 * n * dh * (dm + hk)}
    keys, held = _attended(c)
    flops = 4.0 * d * (hq // hk) * keys
    pair, row = 4 * d, hk * (4 * d + 4)            # K and V of a pair; K, V and logit of a token
    query = hq * (4 * d + 4)                       # q, out and lse of a token
    total, b = sum(_lens(c)), c["batch"]
    if c["kind"] == "soft":
        return {"bytes": total * (row + query), "flops": flops}
    if c["kind"] == "prefill":
        return {"bytes": total * (row + query) + held * pair, "flops": flops}
    if c["kind"] == "feed":
        # the logits of all tokens, the rows that are kept (read, written, read by the decode)
        return {"bytes": total * hk * 4 + 3 * held * pair + b * query,
                "flops": 4.0 * d * (hq // hk) * held}
    n = b * c["tokens"]
    got = {"bytes": held * pair + n * (row + query), "flops": flops}
    if c["kind"] == "predict":
        got["bytes"] += net_bytes + 2 * b * dm
        got["flops"] += 2 * b * dh * (dm + hk)
    return got


def tolerance(case):
    # Measured against exact(): the 32-bit sums of the logits 1.5e-7 (another order of 4096
    # products may show several times that); bf16 rows 2.0e-3 to 2.3e-3, most of it their own
    # rounding, the rest the softmax weights rounded to bf16.  Four times that.
    return {"rel": 2e-6, "max": 2e-4} if case["kind"] == "logits" else {"rel": 9e-3, "max": 0.1}


def _attention(c, q, pos, k, v, f, soft):
    """out and lse of the queries q [n, Hq, D] at positions pos over the rows k, v, f of their
    sequence, in 64 bits: causal, inside the window or gated on (soft: biased by log u)."""
    hk, g, d = c["kv_heads"], c["q_heads"] // c["kv_heads"], c["head_dim"]
    n, t = q.shape[0], k.shape[0]
    out = torch.empty(n, c["q_heads"], d, dtype=torch.float64, device="cuda")
    lse = torch.empty(n, c["q_heads"], dtype=torch.float64, device="cuda")
    step = max(1, (1 << 26) // (g * t))
    for h in range(hk):
        kh, vh = k[:, h].double().t().contiguous(), v[:, h].double().contiguous()
        bias = torch.nn.functional.logsigmoid(f[:, h].double())
        on = f[:, h] >= _theta(c)
        for i in range(0, n, step):
            p = pos[i:i + step, None]
            end = int(pos[min(i + step, n) - 1]) + 1
            age = p - torch.arange(end, device="cuda")[None, :]
            x = (q[i:i + step, h * g:(h + 1) * g].double().reshape(-1, d) @ kh[:, :end]).view(-1, g, end) / math.sqrt(d)
            if soft:
                x += torch.where(age >= c["window"], bias[None, :end], 0.0)[:, None]
                seen = age >= 0
            else:
                seen = (age >= 0) & ((age < c["window"]) | on[None, :end])
            x.masked_fill_(~seen[:, None], -math.inf)
            z = torch.logsumexp(x, dim=-1)
            x = torch.exp(x.sub_(z[..., None]))
            out[i:i + step, h * g:(h + 1) * g] = (x.view(-1, end) @ vh[:end]).view(-1, g, d)
            lse[i:i + step, h * g:(h + 1) * g] = z
    return out, lse


def _logits(net):
    hidden, w1, b1, w2, b2 = (x.double() for x in net)
    x = hidden @ w1.t().contiguous() + b1
    return (x * torch.sigmoid(x)) @ w2.t().contiguous() + b2


def exact(case, seed):
    c = dict(case)
    if c["kind"] == "logits":
        return _logits(_predictor(c, seed, c["tokens"]))
    lens, b = _lens(c), c["batch"]
    size = c["ctx_max"] + 1 if c["kind"] == "soft" else c["tokens"] if c["kind"] in ("prefill", "feed") else 4096
    pieces = list(_prompt(c, seed, size))

    def whole(i, j):                       # input j of sequence i, all pieces
        return torch.cat([p[j][p[3][i]:p[3][i + 1]] for p in pieces])

    n = c["tokens"] if c["kind"] in ("step", "predict", "attend", "score", "chunk") else 0
    new = _new_tokens(c, seed)[0] if n else None
    g = _gen(seed, 3)
    if c["kind"] == "prefill":
        queries = [_query(c, g, p[3][-1]) for p in pieces]
    elif c["kind"] == "soft":
        queries = _query(c, g, pieces[0][3][-1])
    elif c["kind"] == "feed":
        queries = _query(c, g, b)
    got = []
    for i in range(b):
        k, v, f = (whole(i, j) for j in range(3))
        if n:
            k, v, f = (torch.cat([x, y[i * n:(i + 1) * n]]) for x, y in zip((k, v, f), new))
            q, pos = new[4][i * n:(i + 1) * n], torch.arange(lens[i], lens[i] + n)
        elif c["kind"] == "feed":
            q, pos = queries[i:i + 1], torch.tensor([lens[i] - 1])
        else:
            pos = torch.arange(lens[i])
            if c["kind"] == "soft":
                q = queries[pieces[0][3][i]:pieces[0][3][i + 1]]
            else:
                q = torch.cat([x[p[3][i]:p[3][i + 1]] for x, p in zip(queries, pieces)])
        got.append(_attention(c, q, pos.cuda(), k, v, f, c["kind"] == "soft"))
    if c["kind"] == "prefill":             # back to the pieces' packed rows
        at, res = [0] * b, []
        for p in pieces:
            rows = []
            for i in range(b):
                m = p[3][i + 1] - p[3][i]
                rows.append(tuple(x[at[i]:at[i] + m] for x in got[i]))
                at[i] += m
            res.append(tuple(torch.cat([r[j] for r in rows]) for j in range(2)))
        return res
    out, lse = (torch.cat([r[j] for r in got]) for j in range(2))
    return (out, lse, _logits(_predictor(c, seed, b))) if c["kind"] == "predict" else (out, lse)
