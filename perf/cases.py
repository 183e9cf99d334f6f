"""The workloads whose time is tracked, through the package's public entry points.

Every case is one thing a decode loop has the library do: a LoPA iteration
(build, verify, select, commit), one batched verify forward, or the encoding
of a prompt. The model layouts are those of synth.shapes. Two cases run a whole
model (the 2-layer tiny one and the full Dream-7B layout); the others run two
to four decoder layers of a layout, so that a rounding in one layer does not
travel through thirty, with an LM head cut to 16384 tokens, which keeps its
share of the weight bytes near the whole model's.

Weights are drawn so that the residual stream keeps order one: projections
N(0, 1 / fan-in), the two that add to the residual stream scaled by
1 / sqrt(2 layers), embeddings N(0, 1). Prefix K / V rows are N(0, 1), what the
drawn projections give. Tokens are uniform; about half of a block's positions
hold the mask token. The candidate tokens are not among the outputs: on random
weights two correct roundings disagree on a near tie every few hundred rows.
Their probabilities (conf) are.
"""
from __future__ import annotations

import math

import torch

import paper_2512_16229_amd as lp
import synth

TAU = 0.9


# ------------------------------------------------------------------- the cases
def _case(name, op, layout, P, L, k, layers=4, vocab=16384, precision="bf16", causal=0):
    """op: "step" (a LoPA iteration), "forward" (one verify forward of k + 1
    branches of L rows after a prefix of P), "prefill" (encode a P-token prompt
    in blocks of L). causal: the window's block-causal sub-block, 0 for none."""
    return dict(name=name, op=op, layout=layout, P=P, L=L, k=k, layers=layers, vocab=vocab,
                precision=precision, causal=causal)


def listed():
    return [
        # the smallest call: an iteration of the 2-layer model, bound by its launches
        _case("tiny step", "step", "tiny", 64, 16, 3, layers=2, vocab=1024),
        # small model, odd block length and prefix, one lookahead branch
        _case("small ragged forward", "forward", "small128", 37, 7, 1, layers=2, vocab=2048),
        # the headline iteration: whole Dream-7B layout, prefix 512, block 32, k = 7
        _case("dream7b step", "step", "dream7b", 512, 32, 7, layers=28, vocab=152064),
        # a block's first forward (one all-mask branch of 32 rows), paid once per block
        _case("dream7b initial forward", "forward", "dream7b", 512, 32, 0),
        # prompt encoding, a few-shot prompt whose length is no multiple of the block
        _case("dream7b prefill", "prefill", "dream7b", 1000, 32, 7),
        # few branches: the low end of the lookahead settings
        _case("dream7b k3 forward", "forward", "dream7b", 777, 32, 3),
        # many branches over a long prefix (two 256-row tiles)
        _case("dream7b k15 forward", "forward", "dream7b", 2048, 32, 15),
        # multi-head attention layout (no grouping of the query heads)
        _case("llada8b k7 forward", "forward", "llada8b", 1024, 32, 7),
        # the multi-block window: two blocks of 32, block-causal inside the window
        _case("dream7b window forward", "forward", "dream7b", 1500, 64, 7, causal=32),
        # the largest window and verify batch the library takes (2048 rows)
        _case("dream7b wide window forward", "forward", "dream7b", 3000, 256, 7),
        # W8A8 in every projection, and in the MLP alone with few rows
        _case("dream7b fp8 k7 forward", "forward", "dream7b", 512, 32, 7, precision="fp8"),
        _case("llada8b fp8 mlp k1 forward", "forward", "llada8b", 300, 32, 1, precision="fp8_mlp"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    layout = rng.choice(["dream7b", "dream7b", "dream7b", "llada8b", "llada8b", "small128", "tiny"])
    big = layout in ("dream7b", "llada8b")
    vocab = 16384 if big else {"small128": 2048, "tiny": 1024}[layout]
    op = rng.choice(["forward", "forward", "forward", "step", "prefill"])
    precision = rng.choice(["bf16", "bf16", "bf16", "fp8", "fp8_mlp"]) if big else "bf16"
    L = rng.choice([rng.randint(5, 64), rng.randint(5, 64), 16, 32, 32, 64, rng.randint(65, 256)])
    k = 0 if rng.random() < 0.25 else _log_uniform(rng, 1, 15)
    P = _log_uniform(rng, 16, 3000)
    causal = 0
    if op == "prefill":
        L, P = rng.choice([16, 32, 32, 64, rng.randint(17, 64)]), min(P, 1500)
    if op == "step":
        k = min(k, max(1, L // 4))  # enough masked positions for every lookahead branch
    k = min(k, 1024 // L - 1) if big else k
    if op == "forward" and L % 32 == 0 and L > 32 and rng.random() < 0.5:
        causal = 32
    c = _case("", op, layout, P, L, max(k, 0), layers=2, vocab=vocab, precision=precision,
              causal=causal)
    del c["name"]
    return c


# ---------------------------------------------------------------------- inputs
def _cfg(case):
    return synth.config(case["layout"], layers=case["layers"], vocab=case["vocab"])


def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1000003 * (seed + 1) + stream)


def _normal(gen, shape, std):
    return torch.randn(shape, generator=gen, device="cuda", dtype=torch.bfloat16).mul_(std)


def _layer(cfg, seed, i):
    H, F, d = cfg["hidden"], cfg["ffn"], cfg["head_dim"]
    nq, nk = cfg["heads"] * d, cfg["kv_heads"] * d
    g = _gen(seed, 10 + i)
    res = 1.0 / math.sqrt(2 * cfg["layers"])
    w = dict(wq=_normal(g, (nq, H), H ** -0.5), wk=_normal(g, (nk, H), H ** -0.5),
             wv=_normal(g, (nk, H), H ** -0.5), wo=_normal(g, (H, nq), res * nq ** -0.5),
             w_gate=_normal(g, (F, H), H ** -0.5), w_up=_normal(g, (F, H), H ** -0.5),
             w_down=_normal(g, (H, F), res * F ** -0.5))
    for n in ("ln1", "ln2"):
        w[n] = (1 + _normal(g, (H,), 0.1)).contiguous()
    if cfg["qkv_bias"]:
        w.update(bq=_normal(g, (nq,), 0.1), bk=_normal(g, (nk,), 0.1), bv=_normal(g, (nk,), 0.1))
    return w


def _ends(cfg, seed):
    """embedding, final norm, LM head (logits of standard deviation about 1.2)"""
    g = _gen(seed, 1)
    return dict(embed=_normal(g, (cfg["vocab"], cfg["hidden"]), 1.0),
                final_norm=(1 + _normal(g, (cfg["hidden"],), 0.1)).contiguous(),
                lm_head=_normal(g, (cfg["vocab"], cfg["hidden"]), 1.2 * cfg["hidden"] ** -0.5))


def _prefix(cfg, seed, i, P):
    g = _gen(seed, 500 + i)
    shape = (cfg["kv_heads"], P, cfg["head_dim"])
    return _normal(g, shape, 1.0), _normal(g, shape, 1.0)


def _tokens(cfg, case, seed):
    """prompt (prefill), branch rows (forward) or the block's state (step)"""
    g, i32 = _gen(seed, 2), torch.int32
    rand = lambda n: torch.randint(0, cfg["vocab"] - 1, (n,), generator=g, device="cuda").to(i32)
    if case["op"] == "prefill":
        return dict(prompt=rand(case["P"]))
    n = case["L"] * (case["k"] + 1 if case["op"] == "forward" else 1)
    tok = rand(n)
    masked = torch.rand(n, generator=g, device="cuda") < 0.5
    if case["op"] == "forward":
        if case["k"] == 0:
            masked[:] = True  # a block's first forward
        tok[masked] = cfg["mask_id"]
        return dict(branch_tokens=tok)
    # the state before an iteration: positions still masked, their confidence
    # and candidate; three quarters masked so that every branch has a position
    masked = torch.arange(n, device="cuda") >= n // 4
    tok[masked] = cfg["mask_id"]
    conf = torch.rand(n, generator=g, device="cuda")
    conf = torch.where(masked, conf * 0.85, torch.ones_like(conf))
    return dict(tokens=tok, conf=conf, pred=rand(n))


def prepare(case, seed):
    cfg = _cfg(case)
    weights = dict(_ends(cfg, seed), layers=[_layer(cfg, seed, i) for i in range(cfg["layers"])])
    model = lp.Model(cfg, weights, precision=case["precision"])
    del weights
    P, L, nb = case["P"], case["L"], case["k"] + 1
    kv = lp.KV(model, P + 2 * L, nb, L)
    st = dict(case=case, cfg=cfg, model=model, kv=kv, **_tokens(cfg, case, seed))
    if case["op"] == "prefill":
        st["decoder"] = lp.Decoder(model, kv, L, case["k"], TAU)
        return st
    for i in range(cfg["layers"]):
        kv.write(i, 0, *_prefix(cfg, seed, i, P))
    kv.set_block_causal(case["causal"])
    new = lambda n, dtype: torch.empty(n, dtype=dtype, device="cuda")
    st.update(conf_b=new(nb * L, torch.float32), pred_b=new(nb * L, torch.int32))
    if case["op"] == "step":
        i32, f32 = torch.int32, torch.float32
        st.update(branch_tokens=new(nb * L, i32), fill_pos=new(nb, i32), valid=new(nb, torch.uint8),
                  n_valid=new(1, i32), scores=new(nb, f32), winner=new(1, i32),
                  next_tokens=new(L, i32), next_conf=new(L, f32), next_pred=new(L, i32),
                  next_unfilled=new(1, i32), append_offset=new(1, i32))
    return st


# ------------------------------------------------------------------------ pass
def run(st):
    case, model, kv = st["case"], st["model"], st["kv"]
    P, L, nb = case["P"], case["L"], case["k"] + 1
    last = case["layers"] - 1
    if case["op"] == "prefill":
        st["decoder"].prefill(st["prompt"])
        return kv.read(last, 0, P)
    if case["op"] == "step":
        lp.lopa_build_branches(st["tokens"], st["conf"], st["pred"], L, st["cfg"]["mask_id"], TAU,
                               case["k"], st["branch_tokens"], st["fill_pos"], st["valid"],
                               st["n_valid"])
    lp.lopa_verify_forward(model, kv, P, st["branch_tokens"], nb, L, st["conf_b"], st["pred_b"])
    if case["op"] == "forward":
        return st["conf_b"], *kv.read_staging(nb - 1, last, L)
    lp.lopa_branch_confidence_select(st["branch_tokens"], st["conf_b"], st["pred_b"], st["valid"],
                                     nb, L, st["cfg"]["mask_id"], st["scores"], st["winner"],
                                     st["next_tokens"], st["next_conf"], st["next_pred"],
                                     st["next_unfilled"])
    lp.lopa_commit_kv(kv, st["winner"], P, L, st["append_offset"])
    # the branches' rows, not the winner's copies: the winner may be a near tie
    return st["conf_b"], st["scores"], st["branch_tokens"], *kv.read_staging(nb - 1, last, L)


def work(case):
    c = _cfg(case)
    H, F, V, d = c["hidden"], c["ffn"], c["vocab"], c["head_dim"]
    nq, nk, n = c["heads"] * d, c["kv_heads"] * d, c["layers"]
    M = case["P"] if case["op"] == "prefill" else (case["k"] + 1) * case["L"]
    proj = 1 if case["precision"] == "fp8" else 2  # bytes of a QKV / O / LM head weight
    mlp = 2 if case["precision"] == "bf16" else 1
    layer = H * (2 * nq + 2 * nk) * proj + 3 * H * F * mlp
    kv_row = 2 * nk * 2
    if case["op"] == "prefill":
        # block-causal: a block's rows see the prompt up to the block's end; no LM head
        L, P = case["L"], case["P"]
        pairs = sum(min(L, P - b) * min(b + L, P) for b in range(0, P, L))
        return dict(bytes=n * (layer + P * kv_row) + P * (H * 2 + 4) + 2 * P * kv_row,
                    flops=n * (2 * M * (2 * H * (nq + nk) + 3 * H * F) + 4 * pairs * nq))
    kv_bytes = (case["P"] + M) * kv_row + (2 * case["L"] * kv_row if case["op"] == "step" else 0)
    sub = case["causal"]
    own = case["L"] if not sub else (case["L"] + sub) / 2  # mean keys of a row's own block
    return dict(bytes=n * (layer + kv_bytes) + V * H * proj + M * (H * 2 + 12) + 2 * case["L"] * kv_row,
                flops=n * (2 * M * (2 * H * (nq + nk) + 3 * H * F) + 4 * M * (case["P"] + own) * nq)
                + 2 * M * V * H)


def tolerance(case):
    # bf16 operands and fp32 sums: measured 2.1e-3 to 2.7e-3 against 64 bits in
    # every case (1.7e-3 is the rounding of a bf16 K / V row itself). FP8: a
    # last-bit change of an activation moves its E4M3 code by up to 6 %, which
    # the rows that follow carry (0.7e-2 to 4e-2 against 64 bits, which have no
    # bf16 step before the codes).
    if case["precision"] == "bf16":
        return {"rel": 1e-2, "max": 0.1}
    return {"rel": 3e-2, "max": 0.5}


# ---------------------------------------------------------------- 64-bit result
def _norm64(x, w, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * w.double()


def _e4m3(x):
    """x (rows) in E4M3 with a scale per row, as its 64-bit values"""
    amax = x.abs().amax(-1, keepdim=True).clamp_min(1e-300)
    q = (x * (448.0 / amax)).clamp(-448, 448).float().to(torch.float8_e4m3fn)
    return q.double() * (amax / 448.0)


def _linear(x, w, fp8):
    return _e4m3(x) @ _e4m3(w.double()).T if fp8 else x @ w.double().T


def _rope64(x, pos, theta):
    half = x.shape[-1] // 2
    inv = theta ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    ang = pos.double()[:, None] * inv
    c, s = ang.cos(), ang.sin()
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, k, v, seen):
    """q [Hq][n][d], k / v [Hkv][m][d], seen [n][m] or None"""
    rep = q.shape[0] // k.shape[0]
    k, v = k.repeat_interleave(rep, 0), v.repeat_interleave(rep, 0)
    s = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(q.shape[-1])
    if seen is not None:
        s = s.masked_fill(~seen, -math.inf)
    return torch.bmm(torch.softmax(s, -1), v.contiguous())


def exact(case, seed):
    cfg = _cfg(case)
    H, d, Hq, Hkv = cfg["hidden"], cfg["head_dim"], cfg["heads"], cfg["kv_heads"]
    P, L, nb = case["P"], case["L"], case["k"] + 1
    f_all, f_mlp = case["precision"] == "fp8", case["precision"] != "bf16"
    inp, ends = _tokens(cfg, case, seed), _ends(cfg, seed)
    prefill = case["op"] == "prefill"
    if prefill:
        tokens, nb, L, pos0 = inp["prompt"], 1, P, 0
        at = torch.arange(P, device="cuda") // case["L"]
        seen = at[:, None] >= at[None, :]
    else:
        pos0, seen = P, None
        if case["causal"]:
            at = torch.arange(L, device="cuda") // case["causal"]
            seen = torch.cat([torch.ones((L, P), dtype=torch.bool, device="cuda"),
                              at[:, None] >= at[None, :]], 1)
        tokens = inp["branch_tokens"] if case["op"] == "forward" else _branches(cfg, case, inp)
    x = ends["embed"][tokens.long()].double()
    pos = torch.arange(pos0, pos0 + L, device="cuda")
    for i in range(cfg["layers"]):
        w = _layer(cfg, seed, i)
        h = _norm64(x, w["ln1"], cfg["rms_eps"])
        qkv = []
        for n, heads in (("q", Hq), ("k", Hkv), ("v", Hkv)):
            y = _linear(h, w["w" + n], f_all)
            if cfg["qkv_bias"]:
                y = y + w["b" + n].double()
            qkv.append(y.view(nb, L, heads, d).transpose(1, 2))
        q, k, v = _rope64(qkv[0], pos, cfg["rope_theta"]), _rope64(qkv[1], pos, cfg["rope_theta"]), qkv[2]
        out = torch.empty((nb, Hq, L, d), dtype=torch.float64, device="cuda")
        if not prefill:
            pk, pv = (t.double() for t in _prefix(cfg, seed, i, P))
        for b in range(nb):
            kk, vv = (k[b], v[b]) if prefill else (torch.cat([pk, k[b]], 1), torch.cat([pv, v[b]], 1))
            out[b] = _attend(q[b], kk, vv, seen)
        x = x + _linear(out.transpose(1, 2).reshape(nb * L, Hq * d), w["wo"], f_all)
        h = _norm64(x, w["ln2"], cfg["rms_eps"])
        g, u = _linear(h, w["w_gate"], f_mlp), _linear(h, w["w_up"], f_mlp)
        x = x + _linear(g * torch.sigmoid(g) * u, w["w_down"], f_mlp)
    rows = k[nb - 1].contiguous(), v[nb - 1].contiguous()
    if prefill:
        return rows
    logits = _linear(_norm64(x, ends["final_norm"], cfg["rms_eps"]), ends["lm_head"], f_all)
    logits[:, cfg["mask_id"]] = -math.inf
    conf = torch.exp(logits.amax(-1) - torch.logsumexp(logits, -1))
    if case["op"] == "forward":
        return conf, *rows
    open_ = (tokens == cfg["mask_id"]).view(nb, L)
    mean = (conf.view(nb, L) * open_).sum(1) / open_.sum(1)
    return conf, mean, None, *rows


def _branches(cfg, case, inp):
    """The k + 1 branch rows of the step's state: no confidence passes TAU, so
    the most confident masked position fills, and branch j adds the j-th next."""
    masked = inp["tokens"] == cfg["mask_id"]
    order = torch.argsort(torch.where(masked, inp["conf"], -1.0), descending=True, stable=True)
    rows = inp["tokens"].repeat(case["k"] + 1, 1)
    rows[:, order[0]] = inp["pred"][order[0]]
    for j in range(1, case["k"] + 1):
        rows[j, order[j]] = inp["pred"][order[j]]
    return rows.reshape(-1)
