"""Workloads on which the decode library's speed and results are measured.

Three kinds of pass make up a generation service built on the library, and the construction of
the 4-bit river when a model is loaded is the fourth:

  prefill   river_prefill of one prompt, at full depth or at a unified exit depth
  step      river_decode_step of one sequence, one synchronous call per token
  batch     river_decode_batch of several sequences of ragged length and exit depth
  quantize  river_quantize_w4 of one matrix

Shapes are the repository's own configurations (8B shape, 1B shape, tiny fp32, the mid-size shape
of the tests).  Most cases are sections of a few transformer blocks with the LM head cut in the
same proportion; two are whole models.  Tokens are handed over by the caller (as a sampling
program does), so a pass does not depend on how near-ties of the logits fall.

A pass returns what the library computed for the caller to use: logits, hidden states of the
token, similarities and exit positions, and for a prefill the K/V cache rows it wrote.
"""
import math

import numpy as np
import torch

from paper_2604_18396_amd import binding, configs

MATRICES = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down")
MID = configs.ModelConfig("mid-bf16", 3, 1024, 8, 2, 128, 2816, 1002, 500000.0, 1e-5, configs.DTYPE_BF16, 192, 1, 2.0)
SHAPES = {"8b": configs.LLAMA_8B, "1b": configs.LLAMA_1B, "mid": MID, "tiny": configs.TINY}
# the LM head of a section: its share of the whole head for 4 of 32 (8B) and 4 of 16 (1B) blocks
SECTION_VOCAB = {"8b": 16032, "1b": 8000, "mid": 1002, "tiny": 512}
DEV = "cuda:0"


# ------------------------------------------------------------------------------- the cases

def listed():
    def c(name, kind, shape, layers, **kw):
        d = {"name": name, "kind": kind, "shape": shape, "layers": layers, "vocab": SECTION_VOCAB[shape],
             "ffn": SHAPES[shape].d_ffn, "group": 64, "kv_f16": False}
        d.update(kw)
        return d

    return [
        # a short chat turn, not a multiple of any tile; the whole prompt leaves the backbone half way
        c("prefill_8b_77", "prefill", "8b", 4, tokens=77, exit=2),
        # the prompt of the 512-token benchmark workload, at full depth
        c("prefill_8b_512", "prefill", "8b", 4, tokens=512, exit=4),
        # the long prompt of the 4096-token workload, half backbone, half river: the largest prefill
        c("prefill_8b_4096", "prefill", "8b", 4, tokens=4096, exit=2),
        # the 256-token workload's prompt at the 1B shape (head_dim 64), one token short of the tile
        c("prefill_1b_255", "prefill", "1b", 4, tokens=255, exit=4),
        # the headline: one token of the whole 8B-shape model, mean exit depth of the benchmark's schedule
        c("step_8b", "step", "8b", 32, vocab=128256, context=512, exit=18, steps=1, threshold=False),
        # the whole 1B-shape model with Eq. 1 deciding (it fires at the entry layer, well away from a tie)
        c("step_1b", "step", "1b", 16, vocab=32000, context=256, exit=8, steps=1, threshold=True),
        # long context, cache in IEEE half as the paper keeps it
        c("step_8b_long", "step", "8b", 4, context=4096, exit=2, steps=2, threshold=False, kv_f16=True),
        # the smallest call: fp32, one launch per phase, Eq. 1 deciding
        c("step_tiny_fp32", "step", "tiny", 4, context=16, exit=2, steps=4, threshold=True),
        # the 16-sequence workload: ragged lengths around 1024 and ragged exit depths
        c("batch_8b_16", "batch", "8b", 4, context=1024, n_seq=16, exit=2, ragged=True, steps=8),
        # a full batch of short contexts, everybody through the whole backbone
        c("batch_8b_32", "batch", "8b", 4, context=200, n_seq=32, exit=4, ragged=False, steps=8),
        # a nearly idle server: three sequences of the small model
        c("batch_1b_3", "batch", "1b", 4, context=300, n_seq=3, exit=2, ragged=True, steps=8),
        # loading a model: the river twin of the largest matrix of a block
        {"name": "quantize_8b_gate", "kind": "quantize", "rows": 14336, "cols": 4096, "group": 64, "bf16": True},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(("prefill", "step", "batch", "quantize"), (7, 5, 5, 2))[0]
    if kind == "quantize":
        return {"kind": kind, "rows": _log_int(rng, 64, 14336), "cols": 16 * _log_int(rng, 16, 896),
                "group": rng.choice((32, 64, 64, 128)), "bf16": rng.random() < 0.75}
    shape = rng.choice(("8b", "8b", "1b", "mid"))
    if kind == "step" and rng.random() < 0.2:
        shape = "tiny"
    layers = rng.randint(2, 4)
    # feed-forward widths of other models of the size, in steps the kernels' tiles do not divide
    ffn = SHAPES[shape].d_ffn
    if rng.random() < 0.4 and shape != "tiny":
        ffn = 64 * rng.randint(ffn // 128, ffn // 64)
    c = {"kind": kind, "shape": shape, "layers": layers, "vocab": SECTION_VOCAB[shape], "ffn": ffn,
         "group": rng.choice((64, 64, 128)), "kv_f16": shape != "tiny" and rng.random() < 0.3,
         "exit": rng.randint(1, layers)}
    if kind == "prefill":
        c["tokens"] = _log_int(rng, 8, 4096)
    elif kind == "step":
        c["context"] = _log_int(rng, 8, 48) if shape == "tiny" else _log_int(rng, 16, 4096)
        c["steps"] = rng.randint(1, 4)
        c["threshold"] = rng.random() < 0.4
    else:
        c["n_seq"] = rng.randint(2, 32)
        c["context"] = _log_int(rng, 40, 1200)
        c["ragged"] = rng.random() < 0.6
        c["steps"] = rng.randint(2, 8)
    return c


# ------------------------------------------------------------------------------- inputs

def _config(case):
    base = SHAPES[case["shape"]]
    kind = case["kind"]
    n = case["tokens"] if kind == "prefill" else case["context"] + case["steps"] + 2
    # Eq. 1 with tau = 0: the residual stream before and after a block point the same way by a wide
    # margin, so the token leaves at the entry layer, which is then the case's exit position
    threshold = case.get("threshold", False)
    return base.with_(name="case", n_layers=case["layers"], vocab=case["vocab"], d_ffn=case["ffn"], max_seq=n,
                      min_exit_layer=case["exit"] if threshold and case["exit"] < case["layers"] else 1,
                      tau=0.0 if threshold and case["exit"] < case["layers"] else 2.0, river_group=case["group"],
                      kv_dtype=configs.KV_F16 if case["kv_f16"] else configs.KV_SAME)


def _shapes(cfg):
    q, kv, d, f = cfg.n_q_heads * cfg.head_dim, cfg.n_kv_heads * cfg.head_dim, cfg.d_model, cfg.d_ffn
    return {"wq": (q, d), "wk": (kv, d), "wv": (kv, d), "wo": (d, q), "w_gate": (f, d), "w_up": (f, d), "w_down": (d, f)}


def _weights(cfg, seed):
    """Matrices N(0, 0.02^2), norm gains 1 + N(0, 0.1^2), made on the GPU."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    dt = torch.bfloat16 if cfg.dtype == configs.DTYPE_BF16 else torch.float32

    def normal(*shape, mean=0.0, std=0.02):
        return torch.empty(shape, dtype=torch.float32, device=DEV).normal_(mean, std, generator=gen).to(dt)

    w = {"tok_emb": normal(cfg.vocab, cfg.d_model), "lm_head": normal(cfg.vocab, cfg.d_model),
         "final_norm": normal(cfg.d_model, mean=1.0, std=0.1), "layers": []}
    for _ in range(cfg.n_layers):
        blk = {k: normal(*s) for k, s in _shapes(cfg).items()}
        blk["attn_norm"] = normal(cfg.d_model, mean=1.0, std=0.1)
        blk["ffn_norm"] = normal(cfg.d_model, mean=1.0, std=0.1)
        w["layers"].append(blk)
    return w


def _tokens(case, cfg, seed):
    """The prompt of every sequence and the tokens handed to the steps."""
    rng = np.random.default_rng(seed + 1)
    if case["kind"] == "prefill":
        lens, steps = [case["tokens"]], 0
    elif case["kind"] == "step":
        lens, steps = [case["context"]], case["steps"]
    else:
        spread = case["context"] // 4 + 1
        lens, steps = [case["context"] - (37 * b) % spread for b in range(case["n_seq"])], case["steps"]
    prompts = [rng.integers(0, cfg.vocab, size=n, dtype=np.int32) for n in lens]
    return prompts, rng.integers(0, cfg.vocab, size=(steps, len(lens)), dtype=np.int32)


def _exits(case):
    """Exit position of every sequence: the case's, or spread over 1 .. L."""
    n = case.get("n_seq", 1)
    if case.get("ragged", False):
        return [1 + (case["exit"] + 3 * b) % case["layers"] for b in range(n)]
    return [case["exit"]] * n


def _view(ctx, host):
    """The library keeps its results in the caller's workspace and hands them out as host copies:
    the place in the workspace that holds the array `host`, as a tensor (no copy in a pass)."""
    raw = host.contiguous().view(torch.uint8).reshape(-1)
    first = int(raw[:8].view(torch.int64)[0])
    n = raw.numel()
    raw = raw.to(DEV)
    for at in (ctx.workspace[: ctx.workspace_bytes // 256 * 256].view(torch.int64)[::32] == first).nonzero().reshape(-1).tolist():
        part = ctx.workspace[at * 256: at * 256 + n]
        if part.numel() == n and torch.equal(part, raw):
            return part.view(host.dtype).view(host.shape)
    raise RuntimeError("the workspace does not hold this array")


def prepare(case, seed):
    if case["kind"] == "quantize":
        gen = torch.Generator(device=DEV).manual_seed(seed)
        w = torch.empty((case["rows"], case["cols"]), dtype=torch.float32, device=DEV).normal_(0.0, 0.02, generator=gen)
        return {"case": case, "w": w.to(torch.bfloat16) if case["bf16"] else w}
    cfg = _config(case)
    w = _weights(cfg, seed)
    river = binding.quantize_river(cfg, w)
    prompts, tokens = _tokens(case, cfg, seed)
    s = {"case": case, "prompts": prompts, "tokens": tokens, "exits": _exits(case)}
    if case["kind"] == "batch":
        ctx = s["ctx"] = binding.River(cfg, w, river, max_batch=case["n_seq"])
        for b, p in enumerate(prompts):
            ctx.prefill(p, seq=b)
        ctx.decode_batch(case["n_seq"], tokens[0], s["exits"])
        s["logits"] = _view(ctx, torch.from_numpy(ctx.batch_logits()))
        s["hidden"] = _view(ctx, torch.from_numpy(ctx.batch_hidden()))
        return s
    ctx = s["ctx"] = binding.River(cfg, w, river)
    if case["kind"] == "step":
        ctx.prefill(prompts[0])
        ctx.decode_step(int(tokens[0][0]), None if case["threshold"] else case["exit"])
        s["logits"] = _view(ctx, torch.from_numpy(ctx.logits()))
        s["hidden"] = _view(ctx, torch.from_numpy(ctx.hidden()))
        return s
    # a program that serves prompts has served others before this one
    other = np.random.default_rng(seed + 2).integers(0, cfg.vocab, size=case["tokens"], dtype=np.int32)
    ctx.prefill(other, case["exit"])
    store = torch.float16 if case["kv_f16"] else torch.bfloat16 if cfg.dtype == configs.DTYPE_BF16 else torch.float32
    s["k"] = _view(ctx, torch.from_numpy(ctx.kcache()).to(store))
    s["v"] = _view(ctx, torch.from_numpy(ctx.vcache()).to(store))
    s["logits"] = torch.empty(cfg.vocab, dtype=torch.float32, device=DEV)
    return s


# ------------------------------------------------------------------------------- one pass

def run(state):
    case = state["case"]
    if case["kind"] == "quantize":
        codes, scale, zero = binding.river_quantize_w4(state["w"], case["group"])
        return {"codes": codes, "scale": scale, "zero": zero}
    ctx = state["ctx"]
    if case["kind"] == "prefill":
        ctx.prefill(state["prompts"][0], case["exit"], out_logits=state["logits"])
        return {"logits": state["logits"], "k": state["k"], "v": state["v"]}
    if case["kind"] == "step":
        ctx.rewind(case["context"])
        sims, exits = [], []
        for t in state["tokens"]:
            _, e, s = ctx.decode_step(int(t[0]), None if case["threshold"] else case["exit"])
            sims.append(s)
            exits.append(e)
        return {"logits": state["logits"], "hidden": state["hidden"], "sims": np.stack(sims), "exits": np.array(exits)}
    n = case["n_seq"]
    for b, p in enumerate(state["prompts"]):
        ctx.rewind(len(p), b)
    sims, exits = [], []
    for t in state["tokens"]:
        _, e, s = ctx.decode_batch(n, t, state["exits"])
        sims.append(s)
        exits.append(e)
    return {"logits": state["logits"], "hidden": state["hidden"], "sims": np.stack(sims), "exits": np.stack(exits)}


# ------------------------------------------------------------------------------- what a pass needs

def work(case):
    if case["kind"] == "quantize":
        n, es = case["rows"] * case["cols"], 2 if case["bf16"] else 4
        groups = case["rows"] * -(-case["cols"] // case["group"])
        return {"bytes": n * es + n // 2 + 2 * groups * es, "flops": 4 * n}
    cfg = _config(case)
    es = 2 if cfg.dtype == configs.DTYPE_BF16 else 4
    params = sum(r * c for r, c in _shapes(cfg).values())
    groups = sum(r * -(-c // cfg.river_group) for r, c in _shapes(cfg).values())
    dense, twin = params * es, params // 2 + 2 * groups * es
    head = cfg.vocab * cfg.d_model
    kv_row = 2 * cfg.n_kv_heads * cfg.head_dim * es
    qd, L = cfg.n_q_heads * cfg.head_dim, cfg.n_layers
    prompts, tokens = _tokens(case, cfg, 0)
    if case["kind"] == "prefill":
        n, e = case["tokens"], case["exit"]
        return {"bytes": e * dense + (L - e) * twin + head * es + n * (L * kv_row + cfg.d_model * es) + cfg.vocab * 4,
                "flops": 2 * n * params * L + 2 * n * (n + 1) * qd * L + 2 * head}
    total = {"bytes": 0, "flops": 0}
    exits = _exits(case)
    for i in range(case["steps"]):
        seen = sum(len(p) + i + 1 for p in prompts)
        for l in range(1, L + 1):
            total["bytes"] += (dense if any(e >= l for e in exits) else 0) + (twin if any(e < l for e in exits) else 0)
        total["bytes"] += head * es + L * kv_row * seen + len(prompts) * cfg.vocab * 4
        total["flops"] += len(prompts) * 2 * (params * L + head) + 4 * seen * qd * L
    return total


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    if SHAPES[case["shape"]].dtype == configs.DTYPE_F32:
        return {"rel": 2e-6}                    # 3e-7 from 64 bits
    # 16-bit weights and GEMM inputs, rounded K/V: sections are 2e-3 .. 4e-3 from 64 bits, the whole
    # 1B and 8B shapes 4e-3 and 1.1e-2 (a change of rounding travels through 16 and 32 blocks)
    return {"rel": 1.5e-2 if case["layers"] <= 4 else 2e-2 if case["layers"] <= 16 else 3e-2}


# ------------------------------------------------------------------------------- in 64 bits

def _quantized(w, group):
    """4-bit twin of a matrix as the library defines it (32-bit arithmetic, stored scale and zero
    point): (codes, scale, zero), codes unpacked."""
    f = w.float()
    rows, cols = f.shape
    pad = -cols % group
    if pad:
        f = torch.cat([f, f[:, -1:].expand(rows, pad)], 1)
    f = f.view(rows, -1, group)
    mn, mx = f.amin(-1), f.amax(-1)
    scale = torch.where(mx > mn, (mx - mn) / 15.0, torch.ones_like(mx)).to(w.dtype)
    zero = (-mn / scale.float()).to(w.dtype)
    codes = torch.clamp(torch.round(f / scale.float()[..., None] + zero.float()[..., None]), 0, 15)
    return codes, scale, zero


def _twin(w, group):
    codes, scale, zero = _quantized(w, group)
    d = (codes.double() - zero.double()[..., None]) * scale.double()[..., None]
    return d.reshape(w.shape[0], -1)[:, : w.shape[1]]


def _rms(h, gain, eps):
    return h / torch.sqrt(h.square().mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    a = pos.double()[:, None] * base ** (-torch.arange(half, device=DEV, dtype=torch.float64) / half)
    c, s = torch.cos(a)[:, None], torch.sin(a)[:, None]
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, lo * s + hi * c], -1)


def exact(case, seed):
    if case["kind"] == "quantize":
        w = prepare(case, seed)["w"].double()
        rows, cols = w.shape
        pad = -cols % case["group"]
        f = torch.cat([w, w[:, -1:].expand(rows, pad)], 1).view(rows, -1, case["group"])
        mn, mx = f.amin(-1), f.amax(-1)
        scale = torch.where(mx > mn, (mx - mn) / 15.0, torch.ones_like(mx))
        return {"codes": None, "scale": scale, "zero": -mn / scale}
    cfg = _config(case)
    w = _weights(cfg, seed)
    prompts, tokens = _tokens(case, cfg, seed)
    L, nq, nkv, hd = cfg.n_layers, cfg.n_q_heads, cfg.n_kv_heads, cfg.head_dim
    n_seq, steps = len(prompts), len(tokens)
    store = torch.float16 if case["kv_f16"] else torch.bfloat16 if cfg.dtype == configs.DTYPE_BF16 else torch.float32
    # all positions of all sequences as rows: the plain causal transformer, every row through the
    # backbone up to its exit position and through the twins above it
    ids = np.concatenate([np.concatenate([p, tokens[:, b]]) for b, p in enumerate(prompts)])
    lens = [len(p) + steps for p in prompts]
    starts = np.concatenate([[0], np.cumsum(lens)])
    pos = torch.from_numpy(np.concatenate([np.arange(n) for n in lens])).to(DEV)
    in_prompt = torch.from_numpy(np.concatenate([np.arange(n) < n - steps for n in lens])).to(DEV)
    step_rows = torch.tensor([[int(starts[b]) + lens[b] - steps + i for b in range(n_seq)] for i in range(steps)], device=DEV)
    forced = torch.empty(len(ids), dtype=torch.int64, device=DEV)
    for b, e in enumerate(_exits(case)):
        forced[int(starts[b]): int(starts[b + 1])] = e
    if case["kind"] == "prefill":
        exit_of = forced
    else:
        exit_of = torch.where(in_prompt, torch.full_like(forced, L), forced)
        if case.get("threshold", False):
            exit_of = torch.where(in_prompt, exit_of, torch.full_like(forced, L))
    h = w["tok_emb"][torch.from_numpy(ids.astype(np.int64)).to(DEV)].double()
    last = step_rows[-1] if steps else torch.tensor([len(ids) - 1], device=DEV)
    hidden, ks, vs = [h[last]], [], []
    sims = torch.full((steps, n_seq, L), float("nan"), dtype=torch.float64, device=DEV)
    for l in range(L):
        blk = w["layers"][l]
        rows_b, rows_r = exit_of > l, exit_of <= l
        some_b, some_r = bool(rows_b.any()), bool(rows_r.any())

        def lin(x, name):
            out = torch.empty((x.shape[0], blk[name].shape[0]), dtype=torch.float64, device=DEV)
            if some_b:
                out[rows_b] = x[rows_b] @ blk[name].double().t()
            if some_r:
                out[rows_r] = x[rows_r] @ _twin(blk[name], cfg.river_group).t()
            return out

        x = _rms(h, blk["attn_norm"], cfg.rms_eps)
        q = _rope(lin(x, "wq").view(-1, nq, hd), pos, cfg.rope_base)
        k = _rope(lin(x, "wk").view(-1, nkv, hd), pos, cfg.rope_base).to(store)
        v = lin(x, "wv").view(-1, nkv, hd).to(store)
        ks.append(k.reshape(-1, nkv * hd))
        vs.append(v.reshape(-1, nkv * hd))
        o = torch.empty((len(ids), nq, hd), dtype=torch.float64, device=DEV)
        for b in range(n_seq):
            r = slice(int(starts[b]), int(starts[b + 1]))
            mask = pos[r][None, :] > pos[r][:, None]
            for j in range(nq):
                s = q[r, j] @ k[r, j // (nq // nkv)].double().t() / math.sqrt(hd)
                o[r, j] = torch.softmax(s.masked_fill_(mask, -math.inf), -1) @ v[r, j // (nq // nkv)].double()
        h1 = h + lin(o.view(-1, nq * hd), "wo")
        x = _rms(h1, blk["ffn_norm"], cfg.rms_eps)
        h2 = h1 + lin(torch.nn.functional.silu(lin(x, "w_gate")) * lin(x, "w_up"), "w_down")
        if steps:
            a, c = h[step_rows], h2[step_rows]
            s = (a * c).sum(-1) / (a.norm(dim=-1) * c.norm(dim=-1))
            live = rows_b[step_rows]
            sims[:, :, l] = torch.where(live, s, sims[:, :, l])
            if case.get("threshold", False) and cfg.min_exit_layer <= l + 1 < L:
                go = torch.zeros_like(rows_b)
                go[step_rows] = live & (s > cfg.tau)
                exit_of = torch.where(go, torch.full_like(exit_of, l + 1), exit_of)
        h = h2
        hidden.append(h[last])
    logits = _rms(h[last], w["final_norm"], cfg.rms_eps) @ w["lm_head"].double().t()
    hidden = torch.stack(hidden)
    if case["kind"] == "prefill":
        return {"logits": logits[0], "k": torch.stack(ks).float(), "v": torch.stack(vs).float()}
    if case["kind"] == "step":
        return {"logits": logits[0], "hidden": hidden[:, 0], "sims": sims[:, 0].cpu().numpy(), "exits": None}
    return {"logits": logits, "hidden": hidden, "sims": sims.cpu().numpy(), "exits": None}
