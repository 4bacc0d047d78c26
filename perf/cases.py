"""The calls of this framework whose speed is watched: what a decoding program has it do, over the range it is used in.

A case names a model, how many of its layers the engine holds, and one call:
  verify   clasp_verify_forward over `rows` tokens behind a cached prefix (one row = plain decoding)
  draft    clasp_draft_sample: one token through the layers a skip set of `skip` layers keeps
  dp       clasp_dp_select: the layer search with budget `skip` on the states of one verified token
  prefill  clasp_prefill of `rows` prompt tokens, then the cache read out layer by layer with clasp_kv_read, as a
           prompt worker does that hands its cache on
  accept   clasp_spec_accept: the acceptance round of speculative sampling over `rows` drafts

Model sizes are those of the benchmark and test configurations. Weights are random: matrices N(0, 0.02^2), the two that
write into the residual stream scaled by a factor of 0.1 to 1 of each layer's own, since some layers of a trained model
add little (which the layer search is there to find: with one size for all it always skips the last layers); norm gains
around 1, final-norm gains around 3, which spreads the logits as far as a trained model's (a few tokens carry most of the
probability). Cached keys and values are N(0, 1) on the fp16 grid.
"""
import dataclasses
import math
import random

import torch

import paper_2505_24196_amd as clasp

DEVICE = "cuda:0"


@dataclasses.dataclass(frozen=True)
class Shape:
    n_layers: int
    d_model: int
    n_heads: int
    n_kv_heads: int
    head_dim: int
    d_ffn: int
    vocab: int
    dtype: str
    rope_base: float = 500000.0
    rms_eps: float = 1e-5

    @property
    def q_dim(self):
        return self.n_heads * self.head_dim

    @property
    def kv_dim(self):
        return self.n_kv_heads * self.head_dim

    @property
    def elem(self):
        return 4 if self.dtype == "f32" else 2

    def layer_elems(self):
        return self.d_model * (2 * self.q_dim + 2 * self.kv_dim + 3 * self.d_ffn)


MODELS = {
    "tiny-f32": Shape(8, 256, 4, 4, 64, 688, 1024, "f32", 10000.0),
    "small-bf16": Shape(6, 512, 8, 2, 64, 1408, 2064, "bf16"),
    "8b": Shape(32, 4096, 32, 8, 128, 14336, 128256, "bf16"),
    "70b": Shape(80, 8192, 64, 8, 128, 28672, 128256, "bf16"),
}


def listed():
    return [
        # The smallest calls: the fp32 configuration's verify pass (four drafts + the pending token) and layer search,
        # where every kernel takes a few microseconds and launches and latency are the cost.
        dict(name="verify_tiny_f32", call="verify", model="tiny-f32", layers=8, rows=5, prefix=64, logits=True),
        dict(name="dp_tiny_f32", call="dp", model="tiny-f32", layers=8, skip=3, prefix=64, tables=True),
        # A small bf16 model (head_dim 64, two KV heads) behind a ragged prefix, seven rows: a draft length of six.
        dict(name="verify_small_bf16", call="verify", model="small-bf16", layers=6, rows=7, prefix=333, logits=True),
        # The benchmark's own round at the 8B shape, 512 tokens of context, 12 of 32 layers skipped, four drafts: one draft
        # step and the layer search on the whole model ...
        dict(name="draft_8b", call="draft", model="8b", layers=32, skip=12, prefix=512),
        dict(name="dp_8b", call="dp", model="8b", layers=32, skip=12, prefix=512, tables=False),
        # ... and the verify pass, on eight layers so that rounding does not travel through all 32.
        dict(name="verify_8b", call="verify", model="8b", layers=8, rows=5, prefix=512, logits=True),
        # Plain decoding of one row at the longest context of the benchmark's sweep.
        dict(name="decode_8b_long", call="verify", model="8b", layers=8, rows=1, prefix=32768, logits=True),
        # Temperature 1: the acceptance of four drafts over the full vocabulary.
        dict(name="accept_8b", call="accept", model="8b", layers=1, rows=4, temperature=1.0),
        # Prompts: a short question of ragged length, a document of some pages continued after a cached prefix (the second
        # turn of a chat), and a long prompt in one pass.
        dict(name="prefill_8b_short", call="prefill", model="8b", layers=8, rows=300, prefix=0, chunk=384),
        dict(name="prefill_8b_turn", call="prefill", model="8b", layers=8, rows=1100, prefix=1900, chunk=1152),
        dict(name="prefill_8b_long", call="prefill", model="8b", layers=8, rows=4096, prefix=0, chunk=4096),
        # The 70B width: a search with 20 candidates per layer (two row groups of the kernels), with its tables.
        dict(name="dp_70b", call="dp", model="70b", layers=24, skip=20, prefix=1024, tables=True),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    call = rng.choice(("verify", "verify", "verify", "draft", "draft", "dp", "dp", "dp", "prefill", "prefill", "prefill", "accept"))
    if call == "accept":
        return dict(call=call, model=rng.choice(("8b", "8b", "small-bf16")), layers=1, rows=rng.randint(1, 8),
                    temperature=rng.choice((0.7, 1.0, 1.0, 1.3)))
    if call == "prefill":
        model = rng.choice(("8b", "8b", "8b", "small-bf16"))
        rows = _log(rng, 65, 4000)
        chunk = min(4096, (rows + 127) // 128 * 128)
        if rng.random() < 0.2:
            chunk = max(128, chunk // 256 * 128)  # two passes
        return dict(call=call, model=model, layers=rng.randint(3, 7) if model == "8b" else 6, rows=rows,
                    prefix=rng.choice((0, 0, _log(rng, 10, 4000))), chunk=chunk)
    model = rng.choice(("tiny-f32", "small-bf16", "8b", "8b", "8b"))
    if call == "dp" and rng.random() < 0.2:
        model = "70b"
    if model == "tiny-f32":
        layers, prefix = 8, _log(rng, 1, 1000)
    elif model == "small-bf16":
        layers, prefix = 6, _log(rng, 1, 4000)
    elif model == "70b":
        layers, prefix = rng.randint(4, 20), _log(rng, 16, 8000)
    else:
        layers, prefix = rng.randint(4, 20), _log(rng, 16, 32000)
    if call == "verify":
        layers = min(layers, 8)
        return dict(call=call, model=model, layers=layers, rows=rng.choice((1, rng.randint(2, 9), rng.randint(2, 9), rng.randint(10, 32))),
                    prefix=prefix, logits=True)
    if call == "draft":
        return dict(call=call, model=model, layers=layers, skip=rng.randint(1, layers // 2), prefix=prefix)
    return dict(call=call, model=model, layers=layers, skip=rng.randint(1, min(layers - 1, 20)), prefix=prefix, tables=rng.random() < 0.5)


# ---- inputs ------------------------------------------------------------------------------------------------------------
def _generator(seed, stream):
    return torch.Generator(device=DEVICE).manual_seed((seed * 1000003 + stream * 7919 + 1) % (1 << 62))


def _shape(case):
    return dataclasses.replace(MODELS[case["model"]], n_layers=case["layers"])


def _layer_weights(s, seed, layer):
    g = _generator(seed, 100 + layer)
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    dims = {"wq": (s.q_dim, s.d_model), "wk": (s.kv_dim, s.d_model), "wv": (s.kv_dim, s.d_model), "wo": (s.d_model, s.q_dim),
            "w_gate": (s.d_ffn, s.d_model), "w_up": (s.d_ffn, s.d_model), "w_down": (s.d_model, s.d_ffn)}
    scale = 10.0 ** -random.Random(seed * 1000 + layer).random()
    w = {k: torch.empty(r, c, dtype=dt, device=DEVICE).normal_(0.0, 0.02 * (scale if k in ("wo", "w_down") else 1.0), generator=g)
         for k, (r, c) in dims.items()}
    for k in ("attn_norm", "mlp_norm"):
        w[k] = torch.empty(s.d_model, dtype=torch.float32, device=DEVICE).normal_(1.0, 0.1, generator=g)
    return w


def _head(s, seed):
    g = _generator(seed, 1)
    dt = torch.float32 if s.dtype == "f32" else torch.bfloat16
    embed, lm_head = (torch.empty(s.vocab, s.d_model, dtype=dt, device=DEVICE).normal_(0.0, 0.02, generator=g) for _ in range(2))
    return embed, lm_head, torch.empty(s.d_model, dtype=torch.float32, device=DEVICE).normal_(3.0, 0.3, generator=g)


def _prefix(s, seed, layer, n):
    """Keys (rotated) and values of the cached positions 0 .. n-1 of one layer, fp32 [n][n_kv_heads][head_dim]."""
    g = _generator(seed, 10000 + layer)
    return [torch.empty(n, s.n_kv_heads, s.head_dim, dtype=torch.float32, device=DEVICE).normal_(generator=g).half().float() for _ in range(2)]


def _tokens(s, seed, n):
    return torch.randint(0, s.vocab, (n,), generator=_generator(seed, 2), device=DEVICE).to(torch.int32)


def _skip_set(case, seed):
    """The middle layers go first, as they do in practice; which of them differs from seed to seed."""
    layers, skip = case["layers"], case["skip"]
    inner = list(range(1, layers - 1)) if skip <= layers - 2 else list(range(layers))
    chosen = set(random.Random(seed).sample(inner, skip))
    return [1 if l in chosen else 0 for l in range(layers)]


def _accept_inputs(case, s, seed):
    """Logits of the full model, of a draft model near it, the drafts it drew, and the uniform numbers."""
    n, g = case["rows"], _generator(seed, 3)
    p = torch.empty(n + 1, s.vocab, dtype=torch.float32, device=DEVICE).normal_(0.0, 3.5, generator=g)
    q = p[:n] + torch.empty(n, s.vocab, dtype=torch.float32, device=DEVICE).normal_(0.0, 0.3, generator=g)
    drafts = torch.multinomial(torch.softmax(q / case["temperature"], dim=1), 1, generator=g).flatten().to(torch.int32)
    u = torch.randint(0, 1 << 24, (n + 1,), generator=g, device=DEVICE).float() / (1 << 24)
    return p, q, torch.cat([torch.zeros(1, dtype=torch.int32, device=DEVICE), drafts]), u[:n].contiguous(), u[n:].contiguous()


def prepare(case, seed):
    s, call, prefix = _shape(case), case["call"], case.get("prefix", 0)
    rows = case.get("rows", 1)
    most = max(rows + 1, 16) if call in ("verify", "accept") else max(16, case.get("skip", 1))
    engine = clasp.Engine(s, max_seq=(prefix + rows + 63) // 32 * 32, max_rows=min(32, most), device=DEVICE)
    embed, lm_head, final_norm = _head(s, seed)
    engine.set_head(embed, lm_head, final_norm)
    del lm_head
    tokens = _tokens(s, seed, rows)
    x, states = embed[tokens[:1].long()].double(), []
    for l in range(s.n_layers):
        w = _layer_weights(s, seed, l)
        engine.set_layer(l, w)
        if call == "dp":  # the states of the verified token that the search starts from
            states.append(x)
            x = _layer64(s, w, x, _prefix(s, seed, l, prefix), prefix, own=True)
    engine.create()
    for l in range(s.n_layers if prefix else 0):
        engine.clasp_kv_load(l, *_prefix(s, seed, l, prefix))
    st = {"call": call, "engine": engine, "prefix": prefix, "tokens": tokens, "case": case}
    if call == "dp":
        st["states"] = torch.cat(states + [x]).float()
    elif call == "draft":
        st["mask"] = _skip_set(case, seed)
        st["u"] = torch.rand(1, generator=_generator(seed, 3), device=DEVICE)
        st["logits"] = torch.empty(s.vocab, dtype=torch.float32, device=DEVICE)
        st["next"] = torch.empty(1, dtype=torch.int32, device=DEVICE)
    elif call == "accept":
        st["inputs"] = _accept_inputs(case, s, seed)
        st["result"] = torch.empty(2, dtype=torch.int32, device=DEVICE)
    return st


def run(st):
    engine, call, case = st["engine"], st["call"], st["case"]
    if call == "verify":
        return engine.clasp_verify_forward(st["tokens"], st["prefix"], want_hidden=True, want_logits=case["logits"])
    if call == "draft":
        engine.clasp_draft_sample(st["mask"], st["tokens"], st["prefix"], 1.0, st["u"], st["logits"], st["next"])
        return {"logits": st["logits"], "next": st["next"]}
    if call == "dp":
        return engine.clasp_dp_select(st["states"], st["prefix"], case["skip"], want_tables=case["tables"], want_g_final=True)
    if call == "accept":
        p, q, tokens, u_accept, u_final = st["inputs"]
        engine.clasp_spec_accept(p, q, tokens, case["rows"], case["temperature"], u_accept, u_final, st["result"][:1], st["result"][1:])
        return st["result"]
    engine.clasp_prefill(st["tokens"], st["prefix"], case["chunk"])
    return [engine.clasp_kv_read(l, st["prefix"], case["rows"]) for l in range(case["layers"])]


# ---- what one pass cannot do without -------------------------------------------------------------------------------------
def work(case):
    s, call, L, d = _shape(case), case["call"], case["layers"], MODELS[case["model"]].d_model
    n, T = case.get("rows", 1), case.get("prefix", 0)
    if call == "accept":
        return {"bytes": (2 * n + 1) * s.vocab * 4, "flops": 4 * (2 * n + 1) * s.vocab}
    layer, head, kv = s.layer_elems(), s.vocab * d, 2 * T * s.kv_dim * s.elem
    cells = 4 * s.q_dim  # flops of one query row against one cached position
    if call == "verify":
        return {"bytes": (L * layer + head) * s.elem + L * kv + 4 * ((L + 1) * n * d + n * s.vocab),
                "flops": 2 * n * (L * layer + head) + L * n * T * cells}
    if call == "draft":
        k = L - case["skip"]
        return {"bytes": (k * layer + head) * s.elem + k * kv + 4 * s.vocab, "flops": 2 * (k * layer + head) + k * T * cells}
    if call == "dp":
        M = case["skip"]  # a layer sees the candidates that can still reach the last cell
        rows = sum(max(0, min(i - 1, M) - max(1, M - (L - i)) + 1) for i in range(1, L + 1))
        evaluated = sum(min(i - 1, M) >= max(1, M - (L - i)) for i in range(1, L + 1))
        return {"bytes": evaluated * (layer * s.elem + kv) + 4 * (L + 2) * d, "flops": rows * (2 * layer + T * cells)}
    seen = n * T + n * (n + 1) // 2
    last = d * 2 * s.kv_dim  # the last layer ends with its keys and values
    return {"bytes": ((L - 1) * layer + last) * s.elem + (L - 1) * kv + L * 2 * n * s.kv_dim * (s.elem + s.elem + 4),
            "flops": 2 * n * ((L - 1) * layer + last) + (L - 1) * seen * cells}


def tolerance(case):
    """Four times the distance from the 64-bit results that is measured: 3e-7 in fp32; with bf16 weights and 16-bit
    attention operands 4e-4 (small model), 1e-3 behind eight layers and 1.5e-3 behind twenty; 2.1e-3 with the fp16
    activations of long prompt passes."""
    if case["call"] == "accept":
        return "exact"
    if case["model"] == "tiny-f32":
        return {"rel": 2e-6}
    return {"rel": 8e-3 if case["call"] == "prefill" else 4e-3 if case["call"] == "verify" else 6e-3}


# ---- the same results in 64 bits -----------------------------------------------------------------------------------------
def _rms(s, x, gain):
    return x * torch.rsqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * gain.double()


def _rotate(s, x, pos):
    """Half-split rotary embedding of [n][heads][head_dim] at positions `pos` ([n])."""
    half = s.head_dim // 2
    theta = s.rope_base ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    angle = pos.double()[:, None, None] * theta
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * angle.cos() - b * angle.sin(), b * angle.cos() + a * angle.sin()], -1)


def _qkv64(s, w, x, pos):
    h = _rms(s, x, w["attn_norm"])
    q, k, v = (h @ w[m].double().T for m in ("wq", "wk", "wv"))
    n = x.shape[0]
    return (_rotate(s, q.view(n, s.n_heads, s.head_dim), pos), _rotate(s, k.view(n, s.n_kv_heads, s.head_dim), pos),
            v.view(n, s.n_kv_heads, s.head_dim))


def _layer64(s, w, x, prefix, pos0, own=False, keep=None):
    """One layer on the rows x behind a cached prefix: consecutive positions that see each other causally, or (own) every
    row at position pos0 seeing itself only. keep: receives the rows' keys and values."""
    n, T, G = x.shape[0], prefix[0].shape[0], s.n_heads // s.n_kv_heads
    step = torch.arange(n, device=x.device)
    q, k, v = _qkv64(s, w, x, pos0 + (0 * step if own else step))
    if keep is not None:
        keep.extend((k, v))
    blocked = (step[:, None] != step[None, :]) if own else (step[None, :] > step[:, None])
    out = torch.empty_like(q)
    for h in range(s.n_kv_heads):
        kh, vh = torch.cat([prefix[0][:, h].double(), k[:, h]]), torch.cat([prefix[1][:, h].double(), v[:, h]])
        for j in range(h * G, (h + 1) * G):
            score = (q[:, j] @ kh.T) / math.sqrt(s.head_dim)
            score[:, T:].masked_fill_(blocked, -math.inf)
            out[:, j] = torch.softmax(score, -1) @ vh
    a = x + out.view(n, s.q_dim) @ w["wo"].double().T
    h = _rms(s, a, w["mlp_norm"])
    return a + (torch.nn.functional.silu(h @ w["w_gate"].double().T) * (h @ w["w_up"].double().T)) @ w["w_down"].double().T


def _logits64(s, x, head):
    h = _rms(s, x, head[2])
    return torch.cat([h @ part.double().T for part in head[1].split(16384)], 1)


def _cosine(a, b):
    return (a * b).sum(-1) / (a.norm(dim=-1).clamp_min(1e-12) * b.norm(dim=-1).clamp_min(1e-12))


def _search64(case, s, seed):
    """Algorithm 1: per layer all candidates, the better of skipping and computing kept per cell (skipping on ties)."""
    L, M, T = case["layers"], case["skip"], case["prefix"]
    embed = _head(s, seed)[0]
    x = embed[_tokens(s, seed, 1).long()].double()
    x_in = x.float().double()
    scores = torch.full((L + 1, M + 1, 2), math.nan, dtype=torch.float64, device=DEVICE)
    g = [x_in]  # g[j] = g(i, j)
    for i in range(1, L + 1):
        w, prefix = _layer_weights(s, seed, i - 1), _prefix(s, seed, i - 1, T)
        x = _layer64(s, w, x, prefix, T, own=True)
        x_i = x.float().double()
        comp = _layer64(s, w, torch.cat(g[1:]), prefix, T, own=True) if len(g) > 1 else None
        new = [x_i]
        for j in range(1, min(i, M) + 1):
            skip = g[j - 1]
            scores[i, j, 1] = _cosine(x_i, skip)
            if j < len(g):
                cand = comp[j - 1:j]
                scores[i, j, 0] = _cosine(x_i, cand)
                new.append(cand if scores[i, j, 0] > scores[i, j, 1] else skip)
            else:
                new.append(skip)
        g = new
    out = {"mask": None, "g_final": g[M].flatten()}
    if case["tables"]:
        out.update(scores=scores, choice=None)
    return out


def exact(case, seed):
    s, call, T = _shape(case), case["call"], case.get("prefix", 0)
    if call == "accept":
        return None
    if call == "dp":
        return _search64(case, s, seed)
    tokens = _tokens(s, seed, case.get("rows", 1))
    head = _head(s, seed)
    x = head[0][tokens.long()].double()
    mask = _skip_set(case, seed) if call == "draft" else [0] * s.n_layers
    hidden, cache = [x], []
    for l in range(s.n_layers):
        if mask[l]:
            continue
        w = _layer_weights(s, seed, l)
        if call == "prefill" and l == s.n_layers - 1:
            cache.append(_qkv64(s, w, x, T + torch.arange(x.shape[0], device=DEVICE))[1:])
            break
        keep = []
        x = _layer64(s, w, x, _prefix(s, seed, l, T), T, keep=keep)
        if call == "prefill":
            cache.append(keep)
        else:
            hidden.append(x)
    if call == "prefill":
        return cache
    if call == "draft":
        return {"logits": _logits64(s, x, head).flatten(), "next": None}
    return {"argmax": None, "hidden": torch.stack(hidden), "logits": _logits64(s, x, head)}
