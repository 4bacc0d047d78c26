"""Kernels at the sizes where their tilings and dispatch rules end: remainders of a K split, one workgroup too few or too
many, the smallest and largest of a range. Everything goes through the C ABI and is compared with the CPU oracle or a
plain PyTorch float64 evaluation of the same formula."""
import numpy as np
import pytest
import torch

import synth_inputs as si
from oracle import clasp_oracle as oc
from tests.test_gpu_parity import assert_close, oracle_dp_following

pytestmark = pytest.mark.gpu


def build(shape, max_seq, max_rows=32, seed=3):
    import paper_2505_24196_amd as clasp
    model = si.gen_model(shape, seed, "cpu")
    return clasp.Engine(shape, max_seq=max_seq, max_rows=max_rows).load(model), oc.OracleModel(shape, si.model_to_numpy(model))


def verify_against_oracle(shape, row_counts, tol, max_seq=128):
    """Verify passes of the given row counts chained on one cache: all states and logits of every row."""
    eng, om = build(shape, max_seq)
    cache = oc.KVCache(shape, max_seq)
    toks = [int(t) for t in si.gen_tokens(5, sum(row_counts), shape.vocab)]
    pos = 0
    for n in row_counts:
        out = eng.clasp_verify_forward(torch.tensor(toks[pos:pos + n], dtype=torch.int32, device="cuda"), pos,
                                       want_hidden=True, want_logits=True)
        ref = [om.token(t, pos + i, cache, want_states=True) for i, t in enumerate(toks[pos:pos + n])]
        assert_close(out["hidden"].cpu().numpy(), np.stack([r[0] for r in ref], 1), tol, f"{n} rows at {pos}: hidden")
        assert_close(out["logits"].cpu().numpy(), np.stack([r[1] for r in ref]), tol, f"{n} rows at {pos}: logits")
        pos += n
    eng.close()


# The fp32 projections split K/16 steps over eight wavefronts and take them four at a time: K = 48 leaves wavefronts
# without a step, 80 and 272 give unequal slices, 2064 gives several rounds of both stage sets with a remainder. Error of
# one sum of K products: about sqrt(K) * 2^-24 of its size, 2.7e-6 at 2064; four of them per layer, two layers.
@pytest.mark.parametrize("d,heads,kv,hd,ffn", [(48, 3, 1, 16, 80), (272, 17, 17, 16, 48), (256, 4, 2, 64, 2064)])
def test_fp32_projections_with_uneven_k_slices(d, heads, kv, hd, ffn):
    shape = si.ModelShape("edge-f32", 2, d, heads, kv, hd, ffn, 112, "f32")
    verify_against_oracle(shape, (1, 5, 16, 17, 32), 2e-5)


def attention64(q, K, V, pos0):
    """q [n][h][hd], K, V [pos0+n][kv][hd] in float64: row r sees positions 0..pos0+r."""
    n, G = q.shape[0], q.shape[1] // K.shape[1]
    t = torch.arange(pos0 + n)
    out = torch.empty_like(q)
    for r in range(n):
        seen = t <= pos0 + r
        for h in range(q.shape[1]):
            p = torch.softmax((K[seen][:, h // G] @ q[r, h]) / q.shape[2] ** 0.5, 0)
            out[r, h] = p @ V[seen][:, h // G]
    return out


# The fp32 attention takes keys 64 at a time and values in pieces of four positions of 64: no prefix, a piece with 1, 2 or 3
# live positions, one below and above the 64 that are requested up front, several rounds; head_dim below, at and above the
# 64 that are. One layer, so that the hidden state shows the attention: error of the softmax-weighted sum of up to 390
# values and of its scores, each about sqrt(n) * 2^-24, then two projections.
@pytest.mark.parametrize("heads,kv,hd", [(4, 4, 64), (4, 2, 16), (2, 1, 144)])
@pytest.mark.parametrize("T", [0, 1, 62, 63, 64, 65, 387])
def test_fp32_attention_at_the_edges_of_its_pieces(heads, kv, hd, T):
    d = heads * hd
    shape = si.ModelShape("edge-f32-attn", 1, d, heads, kv, hd, 64, 112, "f32")
    eng, om = build(shape, max_seq=448)
    K, V = si.gen_kv(shape, 9, 1, 448, "cpu")
    bad = torch.full((448 - T, kv, hd), float("nan"))  # positions the call may not read
    eng.clasp_kv_load(0, torch.cat([K[0, :T], bad]), torch.cat([V[0, :T], bad]))
    n = 3
    toks = [int(t) for t in si.gen_tokens(5, n, shape.vocab)]
    out = eng.clasp_verify_forward(torch.tensor(toks, dtype=torch.int32, device="cuda"), T, want_hidden=True)
    m = si.gen_model(shape, 3, "cpu")
    w = {k: v.double() for k, v in m["layers"][0].items()}
    x = m["embed"][toks].double()
    rms = lambda v: v * torch.rsqrt((v * v).mean(-1, keepdim=True) + shape.rms_eps)  # noqa: E731
    theta = shape.rope_base ** (-torch.arange(hd // 2, dtype=torch.float64) / (hd // 2))
    ang = (T + torch.arange(n, dtype=torch.float64))[:, None, None] * theta

    def rot(v):
        a, b = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)

    q, k, v = rot((rms(x) @ w["wq"].T).view(n, heads, hd)), rot((rms(x) @ w["wk"].T).view(n, kv, hd)), (rms(x) @ w["wv"].T).view(n, kv, hd)
    att = attention64(q, torch.cat([K[0, :T].double(), k]), torch.cat([V[0, :T].double(), v]), T)
    a = x + att.reshape(n, d) @ w["wo"].T
    y = a + (torch.nn.functional.silu(rms(a) @ w["w_gate"].T) * (rms(a) @ w["w_up"].T)) @ w["w_down"].T
    assert_close(out["hidden"][1].cpu().numpy(), y.numpy(), 2e-5, f"T={T}")
    rk, rv = eng.clasp_kv_read(0, T, n)
    assert_close(rk.cpu().numpy().reshape(n, -1), k.reshape(n, -1).numpy(), 2e-5, "keys")
    assert_close(rv.cpu().numpy().reshape(n, -1), v.reshape(n, -1).numpy(), 2e-5, "values")
    eng.close()


# The last piece of four values that the fp32 attention takes reaches up to three positions beyond the prefix, where the
# values count as zero: a weight multiplied with them has to be a number, also where the launch has no key of its own for it
# (one row behind a prefix of T % 4 = 1 or 2, two rows at 1: plain decoding, drafts, candidates of the search). Every word of
# LDS is a NaN before each call, so a weight that the kernel has not written shows. At the long prefixes those words lie
# beyond what the projections of the same call use of LDS. Error bound as in the test above: the sum of 5000 softmax weights
# adds sqrt(5000) * 2^-24 = 4e-6 of its size.
@pytest.mark.parametrize("T", [1, 2, 3, 4, 61, 62, 63, 5001, 5002, 5003])
def test_fp32_attention_depends_on_no_stale_lds(T):
    from tests.lds_fill import load
    fill = load()
    nan = 0x7fc00000
    shape = si.ModelShape("edge-f32-lds", 3, 256, 4, 2, 64, 64, 112, "f32")
    eng, om = build(shape, max_seq=(T + 32) // 32 * 32 + 32)
    K, V = si.gen_kv(shape, 9, shape.n_layers, T, "cpu")
    for l in range(shape.n_layers):
        eng.clasp_kv_load(l, K[l], V[l])
    toks = [int(t) for t in si.gen_tokens(5, 2, shape.vocab)]
    dtoks = torch.tensor(toks, dtype=torch.int32, device="cuda")

    def prefix():
        cache = oc.KVCache(shape, T + 2)
        cache.load(K.numpy().astype(np.float64), V.numpy().astype(np.float64))
        return cache

    cache = prefix()
    ref = [om.token(t, T + i, cache, want_states=True) for i, t in enumerate(toks)]
    for n in (1, 2):
        fill(nan)
        out = eng.clasp_verify_forward(dtoks[:n], T, want_hidden=True, want_logits=True)
        assert_close(out["hidden"].cpu().numpy(), np.stack([r[0] for r in ref[:n]], 1), 2e-5, f"{n} rows: hidden")
        assert_close(out["logits"].cpu().numpy(), np.stack([r[1] for r in ref[:n]]), 2e-5, f"{n} rows: logits")
    logits, nxt = torch.zeros(shape.vocab, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    fill(nan)
    eng.clasp_draft_sample([0, 1, 0], dtoks[:1], T, 1.0, torch.full((1,), 0.5, device="cuda"), logits, nxt)
    assert_close(logits.cpu().numpy(), om.token(toks[0], T, prefix(), skip=np.array([0, 1, 0]))[1], 2e-5, "draft: logits")
    X = torch.tensor(np.asarray(ref[0][0]), dtype=torch.float32, device="cuda")
    fill(nan)
    gpu = eng.clasp_dp_select(X, T, 2, want_tables=True)
    dp = oracle_dp_following(om, X.cpu().numpy().astype(np.float64), T, prefix(), 2, gpu["choice"].cpu().numpy())
    for k, key in enumerate(("sigma_c", "sigma_s")):
        sc = gpu["scores"].cpu().numpy()[..., k]
        assert np.array_equal(np.isnan(sc), np.isnan(dp[key])) and np.nanmax(np.abs(sc - dp[key])) <= 2e-5, key
    assert_close(gpu["g_final"].cpu().numpy(), dp["g_final"], 2e-5, "g(L, M)")
    eng.close()


# head_dim not a multiple of 8 (fp32 models; matrices handed over as they are, which is what packing does to them): the attention
# goes element by element. Fewer and more rotary pairs than a wavefront has lanes, prefixes up to 109 tokens, LDS full of NaN.
# Bounds as for the projections above.
@pytest.mark.parametrize("heads,kv,hd", [(8, 8, 6), (16, 8, 10), (8, 8, 130)])
def test_fp32_attention_with_odd_head_sizes(heads, kv, hd):
    import paper_2505_24196_amd as clasp
    from tests.lds_fill import load
    fill = load()
    shape = si.ModelShape("edge-f32-odd", 3, 64, heads, kv, hd, 48, 112, "f32")
    model = si.gen_model(shape, 3, "cpu")
    om = oc.OracleModel(shape, si.model_to_numpy(model))
    eng = clasp.Engine(shape, max_seq=128, max_rows=32)
    eng.set_head(model["embed"], model["lm_head"], model["final_norm"])
    for l, w in enumerate(model["layers"]):
        t = {k: v.cuda().contiguous() for k, v in w.items()}
        t["w_gate_up"] = torch.cat([t.pop("w_gate"), t.pop("w_up")])
        eng._layers[l] = t
    eng.create()
    cache = oc.KVCache(shape, 128)
    toks, pos = [int(t) for t in si.gen_tokens(5, 109, shape.vocab)], 0
    for n in (1, 2, 7, 32, 32, 1, 2, 32):
        fill(0x7fc00000)
        out = eng.clasp_verify_forward(torch.tensor(toks[pos:pos + n], dtype=torch.int32, device="cuda"), pos, want_hidden=True, want_logits=True)
        ref = [om.token(t, pos + i, cache, want_states=True) for i, t in enumerate(toks[pos:pos + n])]
        assert_close(out["hidden"].cpu().numpy(), np.stack([r[0] for r in ref], 1), 2e-5, f"{n} rows at {pos}: hidden")
        assert_close(out["logits"].cpu().numpy(), np.stack([r[1] for r in ref]), 2e-5, f"{n} rows at {pos}: logits")
        pos += n
    X = out["hidden"][:, -1].contiguous()
    fill(0x7fc00000)
    gpu = eng.clasp_dp_select(X, pos - 1, 2, want_tables=True)
    dp = oracle_dp_following(om, X.cpu().numpy().astype(np.float64), pos - 1, cache, 2, gpu["choice"].cpu().numpy())
    assert_close(gpu["g_final"].cpu().numpy(), dp["g_final"], 2e-5, "g(L, M)")
    eng.close()


# Draws and acceptance: in one launch (a draw up to 4096 entries, one to four a thread; acceptance up to 1024 entries and seven
# drafts), in two (acceptance up to 4096) and over rows cut into chunks, the last of them of 16 entries, 64 full ones,
# larger than what stays in registers. The mass sits on at most eight tokens, several of them at chunk edges. A running sum of the
# others' weights (e^-39 each) is exact to 1e-7, of the eight and of their fp32 exponentials to 16 * 2^-23 + 8 * 2^-24 = 2.4e-6:
# draws whose uniform number is further than 1e-4 from every float64 running sum have to agree.
@pytest.mark.parametrize("V", [16, 512, 528, 1024, 1040, 2064, 4096, 4112, 8192, 8208, 65536, 128256, 262160])
def test_draws_over_chunk_edges(V):
    import paper_2505_24196_amd as clasp
    shape = si.ModelShape("edge-vocab", 1, 32, 2, 1, 16, 32, V, "f32")
    eng = clasp.Engine(shape, max_seq=32, max_rows=32).load(si.gen_model(shape, 3, "cuda"))
    size = max(1024, (V + 63) // 64)
    hot = sorted({0, 1, size - 1, size, 2 * size, V // 2, V - 2, V - 1} & set(range(V)))
    base = torch.full((V,), -40.0)
    base[hot] = torch.linspace(-1.0, 1.0, len(hot))
    dev = lambda t: t.to("cuda")  # noqa: E731
    tok, acc = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    variants = {"plain": base, "inf": torch.where(base < -30, torch.tensor(-float("inf")), base),
                "lowest": torch.where(base < -30, torch.tensor(torch.finfo(torch.float32).min), base)}
    checked = 0
    for lg in variants.values():
        c = torch.softmax(lg.double() / 0.8, 0).cumsum(0)
        d_lg = dev(lg)
        for u in [0.0, 1 - 2.0 ** -24] + [(i + 0.5) / 23 for i in range(23)]:
            eng.clasp_sample_token(d_lg, 0.8, torch.tensor([u], device="cuda"), tok)
            assert lg[int(tok)] > -30
            if (c - u).abs().min() > 1e-4:
                assert int(tok) == int((c > u).nonzero()[0]), (u, V)
                checked += 1
    assert checked > 40
    for bad in (torch.full((V,), -float("inf")), torch.full((V,), float("nan"))):  # no distribution: -1
        eng.clasp_sample_token(dev(bad), 1.0, torch.tensor([0.5], device="cuda"), tok)
        assert int(tok) == -1
    one_nan = base.clone()
    one_nan[V - 1] = float("nan")
    eng.clasp_sample_token(dev(one_nan), 1.0, torch.tensor([0.5], device="cuda"), tok)
    assert int(tok) == -1
    # acceptance: n drafts, the first rejected one at every place (its draft has probability ~0 under the full model)
    for n in (1, 5, 7, 8, 31):
        for a in sorted({0, n // 2, n - 1, n}):
            p, q = base.repeat(n + 1, 1), base.repeat(n, 1)
            drafts = [hot[i % len(hot)] for i in range(n)]
            if a < n:
                q[a, hot[0]] += 2.0
                p[a, drafts[a]] = -40.0
            u = 0.37
            eng.clasp_spec_accept(dev(p), dev(q), torch.tensor([0] + drafts, dtype=torch.int32, device="cuda"), n, 1.0,
                                  torch.full((n,), 0.5, device="cuda"), torch.tensor([u], device="cuda"), acc, tok)
            w = torch.softmax(p[a].double(), 0)
            if a < n:
                w = (w - torch.softmax(q[a].double(), 0)).clamp_min(0)
            c = w.cumsum(0) / w.sum()
            assert int(acc) == a, (V, n, a)
            if (c - u).abs().min() > 1e-4:
                assert int(tok) == int((c > u).nonzero()[0]), (V, n, a)
    # identical rows and a rejection by u: the residual is empty and the full model's row is drawn from
    p = base.repeat(2, 1)
    eng.clasp_spec_accept(dev(p), dev(base[None]), torch.tensor([0, hot[0]], dtype=torch.int32, device="cuda"), 1, 1.0,
                          torch.full((1,), 1.0, device="cuda"), torch.tensor([0.37], device="cuda"), acc, tok)
    c = torch.softmax(base.double(), 0).cumsum(0)
    assert int(acc) == 0 and int(tok) == int((c > 0.37).nonzero()[0])
    eng.close()


# Prompt passes over every tile, K-split and attention form the launches choose from (tests/test_launches.py holds the shapes and
# row counts below to that, on 256 CUs): row counts at the tiles' edges and remainders, below and above the fp16 threshold
# (640). "cols" has the column counts of the 8B shape's q/k/v and gate/up projections over a short contraction, "rows" those
# of its residual projections over a short one, "odd" an odd number of k-steps everywhere, "one k-step" the shortest
# contraction there is; "wide" is the 8B width itself, whose long contractions take the larger tiles of the residual
# projections in slices, "heads" enough query heads for two tiles per wavefront in the short-prompt attention.
# Reference: the row-limited path on the same tokens, itself held to the oracle elsewhere; the two differ by rounding (fp16
# keys and values, fp16 activations from 640 rows on), the bound is the one every bf16-model result is held to, and a k-step
# or a tile left out or taken twice moves its rows by more (one k-step of the longest contractions, 448: 1/sqrt(448) = 4.7 %).
PROMPT_ROWS = (1, 16, 33, 64, 65, 97, 128, 129, 160, 161, 256, 257, 300, 321, 448, 449, 600, 639, 640, 641, 700, 833, 1000, 1100,
               1537, 2049)
PROMPT_PASSES = {  # kind: (d, heads, kv, hd, ffn), row counts
    "cols": ((256, 32, 8, 128, 14336), PROMPT_ROWS),
    "rows": ((4096, 2, 1, 128, 256), PROMPT_ROWS),
    "odd": ((544, 6, 2, 64, 1440), PROMPT_ROWS),
    "one k-step": ((32, 1, 1, 64, 32), PROMPT_ROWS),
    "wide": ((4096, 32, 8, 128, 14336), (350, 400, 600, 639, 700, 900, 1100, 2048, 3500, 4096)),
    "heads": ((256, 64, 8, 128, 64), (500, 600, 640, 991)),
    "heads 64": ((256, 64, 8, 64, 64), (500, 600, 640, 991)),
}


@pytest.mark.parametrize("kind", PROMPT_PASSES)
def test_prompt_passes_at_the_edges_of_their_tiles(kind):
    import paper_2505_24196_amd as clasp
    (d, heads, kv, hd, ffn), rows = PROMPT_PASSES[kind]
    most = max(rows) + 51
    shape = si.ModelShape("edge-bf16", 3, d, heads, kv, hd, ffn, 2064, "bf16")
    model = si.gen_model(shape, 3, "cuda")
    ref, eng = (clasp.Engine(shape, max_seq=(most + 31) // 32 * 32, max_rows=32).load(model) for _ in range(2))
    toks = si.gen_tokens(5, most, shape.vocab).cuda()
    for s in range(0, most, 30):
        ref.clasp_verify_forward(toks[s:s + 30], s)
    want = [[t.clone() for t in ref.clasp_kv_read(l, 0, most)] for l in range(3)]
    for n in rows:
        eng.clasp_prefill(toks[:n], 0, (n + 127) // 128 * 128)
        for l in range(3):
            for got, full in zip(eng.clasp_kv_read(l, 0, n), want[l]):
                a, b = got.reshape(n, -1), full[:n].reshape(n, -1)
                err = ((a - b).abs().amax(1) / b.abs().amax(1)).max().item()
                assert err <= 2e-2, (kind, n, l, err)
    ref.close()
    eng.close()


# The greedy head over tile counts at the edges of its threads and wavefronts (1, 63, 64, 65, 1024 and 1025 tiles, and more than
# the 8 x 1024 of one round), with gate/up and lm_head on both sides of one workgroup per CU (256 tiles), one and two row
# groups, and a contraction shorter and longer than the wavefronts' first stage. Rows of the row-limited path against the
# oracle; argmax, margin and top-1 probability against the call's own logits (the margin exactly: the same fp32 numbers).
@pytest.mark.parametrize("vocab,d,ffn", [(16, 64, 32), (1008, 64, 2048), (1024, 96, 2080), (1040, 512, 64), (4096, 64, 64),
                                         (4112, 1056, 96), (16384, 64, 64), (16400, 64, 64), (131088, 64, 64)])
def test_greedy_head_and_small_projections(vocab, d, ffn):
    shape = si.ModelShape("edge-head", 2, d, 2, 1, 64, ffn, vocab, "bf16")
    if vocab <= 4112:
        verify_against_oracle(shape, (1, 3, 9, 16, 17, 32), 2e-2)
    import paper_2505_24196_amd as clasp
    eng = clasp.Engine(shape, max_seq=64, max_rows=32).load(si.gen_model(shape, 3, "cuda"))
    for n in (1, 8, 9, 17):
        toks = si.gen_tokens(5, n, vocab).cuda()
        out = eng.clasp_verify_forward(toks, 0, want_logits=True, want_margin=True)
        lg = out["logits"].double()
        top = lg.topk(2, dim=1).values
        assert torch.equal(out["argmax"].long(), lg.argmax(1))
        assert torch.equal(out["margin"].double(), (out["logits"].topk(2, dim=1).values[:, 0] - top[:, 1].float()).double())
    nxt, prob, q = torch.zeros(2, dtype=torch.int32, device="cuda"), torch.zeros(1, device="cuda"), torch.zeros(vocab, device="cuda")
    eng.clasp_draft_step(None, toks[:1], 0, nxt[:1], prob)
    eng.clasp_draft_sample(None, toks[:1], 0, 1.0, torch.zeros(1, device="cuda"), q, nxt[1:])
    assert int(nxt[0]) == int(q.argmax())
    want = torch.softmax(q.double(), 0).max().item()
    assert abs(float(prob) / want - 1) <= 1e-5  # one rescaling and a tree of sums: about 20 roundings of 6e-8
    eng.close()


# Cache contents in and out at the edges of 32-position blocks and 8-position pieces, from and to buffers that are not 16-byte
# aligned: every value comes back exactly, and positions outside the call's range keep what they held.
@pytest.mark.parametrize("dtype,kv,hd", [("bf16", 2, 64), ("bf16", 3, 128), ("f32", 2, 16)])
def test_cache_moves_at_block_edges(dtype, kv, hd):
    import paper_2505_24196_amd as clasp
    shape = si.ModelShape("edge-kv", 2, 64, kv, kv, hd, 64, 112, dtype) if dtype == "bf16" else \
        si.ModelShape("edge-kv", 2, 32, kv, kv, hd, 64, 112, dtype)
    eng = clasp.Engine(shape, max_seq=160, max_rows=4).load(si.gen_model(shape, 3, "cpu"))
    ref = [torch.zeros(160, kv, hd, device="cuda") for _ in range(2)]
    for off in (0, 1):  # element offset of the caller's buffers
        for T in (1, 7, 8, 31, 32, 33, 100, 160):
            bufs = [torch.randn(160 * kv * hd + off, device="cuda").half().float() for _ in range(2)]
            src = [b[off:off + T * kv * hd] for b in bufs]
            rc = clasp.lib().clasp_kv_load(eng._ctx, 1, src[0].data_ptr(), src[1].data_ptr(), T, None)
            assert rc == 0
            torch.cuda.synchronize()
            for r, s in zip(ref, src):
                r[:T] = s.view(T, kv, hd)
            for pos0, n in ((0, 160), (T - 1, 161 - T), (5, 29), (32, 32), (40, 1), (63, 66)):
                n = min(n, 160 - pos0)
                out = [torch.full((160 * kv * hd + off + 64,), -7.0, device="cuda") for _ in range(2)]
                rc = clasp.lib().clasp_kv_read(eng._ctx, 1, pos0, n, out[0].data_ptr() + 4 * off, out[1].data_ptr() + 4 * off, None)
                assert rc == 0
                torch.cuda.synchronize()
                for o, r in zip(out, ref):
                    assert torch.equal(o[off:off + n * kv * hd].view(n, kv, hd), r[pos0:pos0 + n]), (off, T, pos0, n)
                    assert (o[:off] == -7).all() and (o[off + n * kv * hd:] == -7).all()
    assert all((t == 0).all() for t in eng.clasp_kv_read(0, 0, 160))  # the other layer
    eng.close()
