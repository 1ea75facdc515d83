"""Timed cases of the serving step, each through a public entry point.

Two cases serve whole workloads through ``lp.Engine`` (the fp32 tiny model and
a full-width 8B-shape model of four layers) and return logits.  The others are
the layers such a run is made of, called one by one on caller-owned buffers:
the projections of decode and prefill steps, the RMSNorm with its residual
fold, attention over the paged cache in both phases, and the token choice.

Sizes come from the model shapes in ``synth.SHAPES`` and from the request
lengths of ``synth.WORKLOADS`` (lognormal prompts of 16 to 4,096 tokens, up to
64 running requests).  ``draw`` spreads over the same ranges.
"""
import math
import random

import numpy as np
import torch

from paper_2410_02425_amd import lp, synth

DEV = "cuda"
DTYPES = {"f16": torch.float16, "bf16": torch.bfloat16}


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest service there is: the fp32 model, four users, short
        # prompts; every step is a chain of small launches
        dict(name="serve tiny fp32", kind="serve_tiny", requests=4, in_len=32, out_len=16),
        # a running batch of an 8B-shape service with mixed prompt and output
        # lengths, prefill and decode steps of the bf16 model as deployed
        dict(name="serve 8b 4 layers", kind="serve", model="8b", layers=4, requests=24, in_mean=400, out_max=24),
        # one user decoding alone: the output projection on a single row
        dict(name="decode o 1 row", kind="gemm", model="7b", proj="o", rows=1, dtype="f16"),
        # a full decode batch: the largest projection of a layer on 64 rows
        dict(name="decode gate/up 64 rows", kind="gemm", model="8b", proj="gu", rows=64, dtype="f16"),
        # a typical prompt's prefill step: a long contraction over few tiles
        dict(name="prefill down 553 rows", kind="gemm", model="8b", proj="down", rows=553, dtype="f16"),
        # a packed prefill of many prompts (or one long one), bf16 inputs
        dict(name="prefill gate/up 4223 rows", kind="gemm", model="8b", proj="gu", rows=4223, dtype="bf16"),
        # the norm between two projections of a prefill step, folding the
        # split-K partials of the first into the residual stream
        dict(name="norm 553 rows 3 partials", kind="norm", rows=553, d=4096, parts=3, dtype="f16"),
        # decode attention of a full batch with the workload's mixed contexts
        dict(name="decode attention 64 rows", kind="decode_attn", model="8b", rows=64, ctx_mean=600, dtype="f16"),
        # a few long conversations on the largest shape (8 query heads a KV head)
        dict(name="decode attention 3 long rows", kind="decode_attn", model="70b", rows=3, ctx_mean=3000,
             dtype="bf16"),
        # the attention of one typical prompt, of odd length
        dict(name="prefill attention 547", kind="prefill_attn", model="8b", prompts=1, len_mean=547, dtype="f16"),
        # the attention of a step of long prompts
        dict(name="prefill attention 3 long", kind="prefill_attn", model="8b", prompts=3, len_mean=2100,
             dtype="bf16"),
        # the next tokens of a full batch whose requests carry different
        # decoding parameters (greedy, temperature, top-k, top-p)
        dict(name="sample 64 rows", kind="sample", model="8b", rows=64, mix="all"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["serve_tiny", "serve", "gemm_decode", "gemm_decode", "gemm_prefill", "gemm_prefill", "norm",
                       "decode_attn", "decode_attn", "prefill_attn", "prefill_attn", "sample"])
    dtype = rng.choice(["f16", "f16", "bf16"])
    if kind == "serve_tiny":
        return dict(kind=kind, requests=rng.randint(1, 12), in_len=rng.randint(5, 100), out_len=rng.randint(4, 16))
    if kind == "serve":
        return dict(kind=kind, model="8b", layers=rng.choice([2, 3, 4]), requests=_log_int(rng, 1, 24),
                    in_mean=_log_int(rng, 60, 400), out_max=rng.randint(4, 24))
    if kind == "gemm_decode":
        return dict(kind="gemm", model=rng.choice(["7b", "8b", "13b", "70b"]),
                    proj=rng.choice(["qkv", "o", "gu", "down", "head"]), rows=_log_int(rng, 1, 64), dtype=dtype)
    if kind == "gemm_prefill":
        while True:
            c = dict(kind="gemm", model=rng.choice(["7b", "8b", "13b", "70b"]),
                     proj=rng.choice(["qkv", "o", "gu", "down"]), rows=_log_int(rng, 65, 4223), dtype=dtype)
            n, k = _proj(c["model"], c["proj"])
            if c["rows"] * n * k <= 4223 * 28672 * 4096:
                return c
    if kind == "norm":
        return dict(kind=kind, rows=_log_int(rng, 1, 2000), d=rng.choice([4096, 5120, 8192]),
                    parts=rng.choice([0, 2, 3, 5, 8]), dtype=dtype)
    if kind == "decode_attn":
        return dict(kind=kind, model=rng.choice(["7b", "8b", "13b", "70b"]), rows=_log_int(rng, 1, 64),
                    ctx_mean=_log_int(rng, 60, 800), dtype=dtype)
    if kind == "prefill_attn":
        prompts = rng.choice([1, 1, 2, 3, 6])
        return dict(kind=kind, model=rng.choice(["7b", "8b", "13b"]), prompts=prompts,
                    len_mean=_log_int(rng, 40, 2100 if prompts <= 3 else 700), dtype=dtype)
    return dict(kind="sample", model=rng.choice(["7b", "8b"]), rows=_log_int(rng, 1, 64),
                mix=rng.choice(["all", "top_p", "top_k", "temperature"]))


# ------------------------------------------------------------------ shapes

def _proj(model, proj):
    """(N, K) of a projection."""
    s = synth.SHAPES[model]
    hd = s.d_model // s.n_heads
    return {"qkv": ((s.n_heads + 2 * s.n_kv_heads) * hd, s.d_model), "o": (s.d_model, s.d_model),
            "gu": (2 * s.ffn_dim, s.d_model), "down": (s.d_model, s.ffn_dim), "head": (s.vocab, s.d_model)}[proj]


def _decode_splits(proj, n, k):
    """K splits a decode step asks for: at most 2,048 16-column slices times
    splits, at least 512 of K each; gate/up and the head are not split."""
    if proj in ("gu", "head"):
        return 1
    return max(1, min(2048 // max(1, n // 16), k // 512))


def _lengths(case, n, mean, hi):
    """n lognormal lengths around `mean`, a function of the case alone."""
    rng = random.Random("%s %d %d" % (case.get("model"), n, mean))
    return [max(1, min(hi, int(round(mean * math.exp(rng.gauss(0.0, 0.5)))))) for _ in range(n)]


def _serve_lengths(case):
    ins = _lengths(case, case["requests"], case["in_mean"], 4 * case["in_mean"])
    outs = [max(2, case["out_max"] - 3 * (i % 5)) for i in range(case["requests"])]
    return ins, outs


def _gen(seed, salt=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed * 16 + salt)
    return g


def _randn(shape, gen, scale=1.0, dtype=torch.float32):
    return (torch.randn(shape, generator=gen, device=DEV) * scale).to(dtype)


# ------------------------------------------------------------------ prepare

class _Req:
    def __init__(self, rid, prompt, out_len):
        self.id, self.prompt, self.out_len, self.arrival_ns = rid, prompt, out_len, 0


def _tiny_weights(seed):
    """Canonical tensors of the tiny model, fp32 (gains 1, weights N(0, 0.02^2))."""
    s = synth.SHAPES["tiny"]
    rng = np.random.default_rng(seed)
    d, f = s.d_model, s.ffn_dim
    kv = s.n_kv_heads * (d // s.n_heads)
    shapes = [(s.vocab, d)]
    for _ in range(s.n_layers):
        shapes += [(d,), (d, d), (kv, d), (kv, d), (d, d), (d,), (f, d), (f, d), (d, f)]
    shapes += [(d,), (s.vocab, d)]
    return [np.ones(x, np.float32) if len(x) == 1 else (rng.standard_normal(x) * 0.02).astype(np.float32)
            for x in shapes]


def _tiny_requests(case, seed):
    rng = np.random.default_rng(seed + 1)
    v = synth.SHAPES["tiny"].vocab
    reqs = [_Req(i, rng.integers(0, v, case["in_len"], dtype=np.int32), case["out_len"])
            for i in range(case["requests"])]
    forced = [rng.integers(0, v, case["out_len"] - 1, dtype=np.int32) for _ in reqs]
    return reqs, forced


def _engine_state(eng, reqs, forced, rows):
    eng.submit(reqs)
    for r, f in zip(reqs, forced):
        eng.set_forced_tokens(r.id, f)
    return {"run": _run_engine, "engine": eng, "reqs": reqs, "rows": rows}


def _prepare_serve_tiny(case, seed):
    s = synth.SHAPES["tiny"]
    reqs, forced = _tiny_requests(case, seed)
    opt = lp.EngineOptions(min(case["requests"], 8), 128, 0, 4096, 0, lp.LP_FLAG_KEEP_LOGITS)
    eng = lp.Engine(lp.make_config(s), opt)
    eng.load_weights(b"".join(w.tobytes() for w in _tiny_weights(seed)))
    return _engine_state(eng, reqs, forced, "all")


def _prepare_serve(case, seed):
    s = synth.SHAPES[case["model"]]
    ins, outs = _serve_lengths(case)
    rng = np.random.default_rng(seed)
    reqs = [_Req(i, rng.integers(0, s.vocab, n, dtype=np.int32), m) for i, (n, m) in enumerate(zip(ins, outs))]
    forced = [rng.integers(0, s.vocab, m - 1, dtype=np.int32) for m in outs]
    opt = lp.EngineOptions(case["requests"], max(a + b for a, b in zip(ins, outs)), 0, max(sum(ins), 64), 0,
                           lp.LP_FLAG_KEEP_LOGITS)
    eng = lp.Engine(lp.make_config(s, n_layers=case["layers"]), opt)
    eng.init_weights_random(seed)
    return _engine_state(eng, reqs, forced, "ends")


def _run_engine(st):
    # tokens are forced, so that one rounding does not change what follows;
    # the logits are what the greedy choice of each step was taken from
    eng = st["engine"]
    eng.run(lp.LP_CLOSED_LOOP, len(st["reqs"]))
    out = []
    for r in st["reqs"]:
        ks = range(r.out_len) if st["rows"] == "all" else (0, r.out_len - 1)
        out.append(np.stack([eng.logits(r.id, k) for k in ks]))
    return out


def _gemm_inputs(case, seed):
    n, k = _proj(case["model"], case["proj"])
    g = _gen(seed)
    x = _randn((case["rows"], k), g, dtype=DTYPES[case["dtype"]])
    w = _randn((n, k), g, 0.02, DTYPES[case["dtype"]])
    return x, w


def _prepare_gemm(case, seed):
    x, w = _gemm_inputs(case, seed)
    (n, k), m = w.shape, case["rows"]
    packed = torch.empty(lp.packed_weight_elems(n, k), dtype=w.dtype, device=DEV)
    lp.op_pack_weight(w, packed)
    splits = lp.op_gemm_plan(m, n, k, 0)[2] if m > 64 else _decode_splits(case["proj"], n, k)
    ws = torch.empty(splits * m * n if splits > 1 else 1, dtype=torch.float32, device=DEV)
    y = torch.empty(m, n, dtype=torch.float32, device=DEV)
    return {"run": _run_gemm, "x": x, "w": packed, "y": y, "ws": ws, "n": n, "splits": splits}


def _run_gemm(st):
    lp.op_gemm(st["x"], st["w"], st["y"], st["splits"], st["ws"], N=st["n"])
    return st["y"]


def _norm_inputs(case, seed):
    g = _gen(seed)
    rows, d = case["rows"], case["d"]
    x = _randn((rows, d), g)
    part = _randn((case["parts"], rows, d), g, 0.05) if case["parts"] else None
    gain = 1.0 + _randn((d,), g, 0.1)
    return x, part, gain


def _prepare_norm(case, seed):
    x, part, gain = _norm_inputs(case, seed)
    y = torch.empty(case["rows"], case["d"], dtype=DTYPES[case["dtype"]], device=DEV)
    return {"run": _run_norm, "x": x, "part": part, "g": gain, "y": y, "parts": case["parts"]}


def _run_norm(st):
    lp.op_rmsnorm(st["x"], st["g"], st["y"], 1e-5, st["part"], st["parts"])
    return [st["x"], st["y"]]


def _heads(model):
    s = synth.SHAPES[model]
    return s.n_heads, s.n_kv_heads, s.d_model // s.n_heads


def _paged_cache(lens, hkv, hd, dtype, gen, seed):
    """A pool of 64-token blocks, each sequence's blocks scattered over it."""
    nb = [-(-n // 64) for n in lens]
    total = sum(nb) + 5
    kc = _randn((total, hkv, 64, hd), gen, dtype=dtype)
    vc = _randn((total, hkv, hd, 64), gen, dtype=dtype)
    perm = np.random.default_rng(seed).permutation(total).astype(np.int32)
    bt = np.zeros((len(lens), max(nb)), dtype=np.int32)
    at = 0
    for i, n in enumerate(nb):
        bt[i, :n] = perm[at:at + n]
        at += n
    return kc, vc, bt


def _decode_inputs(case, seed):
    hq, hkv, hd = _heads(case["model"])
    ctx = _lengths(case, case["rows"], case["ctx_mean"], 4096)
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    kc, vc, bt = _paged_cache(ctx, hkv, hd, dt, g, seed)
    q = _randn((case["rows"], hq, hd), g, dtype=dt)
    return ctx, q, kc, vc, bt


def _prepare_decode_attn(case, seed):
    ctx, q, kc, vc, bt = _decode_inputs(case, seed)
    m, hq, hd = q.shape
    ws = torch.empty(lp.decode_attention_ws_bytes(m, hq, hd, max(ctx)) // 4 + 1, dtype=torch.float32, device=DEV)
    return {"run": _run_decode_attn, "q": q, "out": torch.empty_like(q), "k": kc, "v": vc,
            "bt": torch.from_numpy(bt).to(DEV), "slot": torch.arange(m, dtype=torch.int32, device=DEV),
            "pos": torch.tensor([c - 1 for c in ctx], dtype=torch.int32, device=DEV), "hkv": kc.shape[1],
            "max_ctx": max(ctx), "ws": ws}


def _run_decode_attn(st):
    lp.op_decode_attention(st["q"], st["out"], st["k"], st["v"], st["bt"], st["slot"], st["pos"], st["hkv"],
                           st["max_ctx"], st["ws"])
    return st["out"]


def _prefill_lengths(case):
    if case["prompts"] == 1:
        return [case["len_mean"]]
    return _lengths(case, case["prompts"], case["len_mean"], min(4096, 2 * case["len_mean"]))


def _prefill_inputs(case, seed):
    hq, hkv, hd = _heads(case["model"])
    lens = _prefill_lengths(case)
    g, dt = _gen(seed), DTYPES[case["dtype"]]
    kc, vc, bt = _paged_cache(lens, hkv, hd, dt, g, seed)
    q = _randn((sum(lens), hq, hd), g, dtype=dt)
    return lens, q, kc, vc, bt


def _prepare_prefill_attn(case, seed):
    lens, q, kc, vc, bt = _prefill_inputs(case, seed)
    start = torch.tensor(np.concatenate([[0], np.cumsum(lens)]), dtype=torch.int32, device=DEV)
    return {"run": _run_prefill_attn, "q": q, "out": torch.empty_like(q), "k": kc, "v": vc,
            "bt": torch.from_numpy(bt).to(DEV), "start": start,
            "slot": torch.arange(len(lens), dtype=torch.int32, device=DEV), "max_len": max(lens),
            "hkv": kc.shape[1]}


def _run_prefill_attn(st):
    lp.op_prefill_attention(st["q"], st["out"], st["k"], st["v"], st["bt"], st["start"], st["slot"], st["max_len"],
                            st["hkv"])
    return st["out"]


# (temperature, top_k, top_p) of requests as services see them
SAMPLING = {"greedy": (0.0, 0, 1.0), "temperature": (1.0, 0, 1.0), "top_k": (0.7, 40, 1.0),
            "top_p": (1.0, 0, 0.9), "both": (0.8, 50, 0.95)}


def _prepare_sample(case, seed):
    v = synth.SHAPES[case["model"]].vocab
    g = _gen(seed)
    # logits of a trained model: a broad body and a few likely tokens per row
    logits = _randn((case["rows"], v), g, 2.0)
    top = torch.randint(0, v, (case["rows"], 24), generator=g, device=DEV)
    logits.scatter_add_(1, top, _randn(top.shape, g, 4.0).abs())
    names = ["greedy", "temperature", "top_k", "top_p", "both"] if case["mix"] == "all" else [case["mix"]]
    rng = random.Random(seed)
    rows = []
    for i in range(case["rows"]):
        t, k, p = SAMPLING[names[i % len(names)]]
        rows.append((t, k, p, (rng.getrandbits(32), rng.getrandbits(32)), (i, 0, rng.randrange(1000))))
    return {"run": _run_sample, "logits": logits, "prm": torch.from_numpy(lp.sample_params_array(rows)).to(DEV),
            "tok": torch.empty(case["rows"], dtype=torch.int32, device=DEV)}


def _run_sample(st):
    lp.op_sample(st["logits"], st["prm"], st["tok"])
    return st["tok"]


PREPARE = {"serve_tiny": _prepare_serve_tiny, "serve": _prepare_serve, "gemm": _prepare_gemm, "norm": _prepare_norm,
           "decode_attn": _prepare_decode_attn, "prefill_attn": _prepare_prefill_attn, "sample": _prepare_sample}


def prepare(case, seed):
    return PREPARE[case["kind"]](case, seed)


def run(state):
    return state["run"](state)


# ------------------------------------------------------------------ work, tolerance

def _serve_work(s, layers, ins, outs, max_batch, esz):
    """One prefill of every prompt, then decode steps that read the weights
    once each and every row's cache; the embedding table is gathered."""
    hd = s.d_model // s.n_heads
    kv = 2 * s.n_kv_heads * hd * esz
    qkv = (s.n_heads + 2 * s.n_kv_heads) * hd
    w = layers * (s.d_model * qkv + s.d_model * s.d_model + 3 * s.d_model * s.ffn_dim)
    head = s.vocab * s.d_model
    waves = -(-len(ins) // max_batch)
    steps = waves * (max(outs) - 1)
    ctx = sum(sum(a + j for j in range(1, b)) for a, b in zip(ins, outs))
    toks = sum(outs)
    nbytes = (steps + waves) * (w + head) * esz + layers * kv * (ctx + 2 * sum(ins)) + toks * s.vocab * 4
    flops = 2 * w * (sum(ins) + toks) + 2 * head * toks
    flops += layers * 4 * s.n_heads * hd * (sum(n * (n + 1) // 2 for n in ins) + ctx)
    return {"bytes": nbytes, "flops": flops}


def work(case):
    k = case["kind"]
    if k == "serve_tiny":
        n = case["requests"]
        s = synth.SHAPES["tiny"]
        return _serve_work(s, s.n_layers, [case["in_len"]] * n, [case["out_len"]] * n, min(n, 8), 4)
    if k == "serve":
        ins, outs = _serve_lengths(case)
        return _serve_work(synth.SHAPES[case["model"]], case["layers"], ins, outs, case["requests"], 2)
    if k == "gemm":
        n, kk = _proj(case["model"], case["proj"])
        m = case["rows"]
        return {"bytes": 2 * (n * kk + m * kk) + 4 * m * n, "flops": 2 * m * n * kk}
    if k == "norm":
        e = case["rows"] * case["d"]
        # without partials the residual stream is only read
        return {"bytes": e * (4 * (1 + case["parts"]) + (4 if case["parts"] else 0) + 2) + 4 * case["d"],
                "flops": e * (4 + case["parts"])}
    if k == "decode_attn":
        hq, hkv, hd = _heads(case["model"])
        ctx = sum(_lengths(case, case["rows"], case["ctx_mean"], 4096))
        return {"bytes": ctx * hkv * hd * 4 + case["rows"] * hq * hd * 4, "flops": 4 * ctx * hq * hd}
    if k == "prefill_attn":
        hq, hkv, hd = _heads(case["model"])
        lens = _prefill_lengths(case)
        return {"bytes": sum(lens) * (hkv * hd * 4 + hq * hd * 4),
                "flops": sum(2 * n * (n + 1) for n in lens) * hq * hd}
    v = synth.SHAPES[case["model"]].vocab
    return {"bytes": case["rows"] * v * 4, "flops": case["rows"] * v * 4}


def tolerance(case):
    k = case["kind"]
    if k == "sample":
        return "exact"  # token ids
    if k == "gemm":
        return {"rel": 5e-6}  # exact products, 32-bit sums
    if k == "serve_tiny":
        return {"rel": 1e-5}  # 32-bit throughout
    if k == "serve":
        return {"rel": 1e-2}  # 16-bit activations through every layer
    if k == "norm":
        return {"rel": 1e-3 if case["dtype"] == "f16" else 8e-3}
    return {"rel": 1.5e-3 if case["dtype"] == "f16" else 1.2e-2}  # 16-bit weights of V and outputs


# ------------------------------------------------------------------ results in 64 bits

def _attend64(q, k, v, first):
    """q [n, Hq, hd] at positions first.., k, v [ctx, Hkv, hd], in float64."""
    n, hq, hd = q.shape
    ctx, hkv, _ = k.shape
    out = torch.empty(n, hq, hd, dtype=torch.float64, device=q.device)
    pos = torch.arange(first, first + n, device=q.device)[:, None]
    late = torch.arange(ctx, device=q.device)[None, :] > pos
    for h in range(hq):
        g = h // (hq // hkv)
        sc = (q[:, h].double() @ k[:, g].double().t().contiguous()) / math.sqrt(hd)
        out[:, h] = torch.softmax(sc.masked_fill(late, -math.inf), dim=1) @ v[:, g].double().contiguous()
    return out


def _sequence(kc, vc, blocks, n):
    """K and V [n, Hkv, hd] of one sequence out of the paged cache."""
    b = torch.from_numpy(blocks[: -(-n // 64)].astype(np.int64)).to(kc.device)
    k = kc[b].permute(0, 2, 1, 3).reshape(-1, kc.shape[1], kc.shape[3])[:n]
    v = vc[b].permute(0, 3, 1, 2).reshape(-1, vc.shape[1], vc.shape[2])[:n]
    return k, v


def _norm64(x, eps):
    return x / torch.sqrt((x * x).mean(dim=1, keepdim=True) + eps)


def _tiny64(weights, tokens):
    """Logits of every position of one token sequence, float64 on the host."""
    s = synth.SHAPES["tiny"]
    hd, n = s.d_model // s.n_heads, len(tokens)
    w = [torch.from_numpy(x).double() for x in weights]
    x = w[0][torch.from_numpy(np.asarray(tokens, dtype=np.int64))]
    theta = float(s.rope_theta) ** (-torch.arange(hd // 2, dtype=torch.float64) * 2 / hd)
    ang = torch.arange(n, dtype=torch.float64)[:, None] * theta[None, :]
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]

    def rope(t):
        a, b = t[..., : hd // 2], t[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], dim=-1)

    for layer in range(s.n_layers):
        an, wq, wk, wv, wo, mn, wg, wu, wd = w[1 + 9 * layer: 10 + 9 * layer]
        h = _norm64(x, s.norm_eps) * an
        q, k, v = (t.reshape(n, -1, hd) for t in (h @ wq.t(), h @ wk.t(), h @ wv.t()))
        x = x + _attend64(rope(q), rope(k), v, 0).reshape(n, -1) @ wo.t()
        h = _norm64(x, s.norm_eps) * mn
        x = x + (torch.nn.functional.silu(h @ wg.t()) * (h @ wu.t())) @ wd.t()
    return (_norm64(x, s.norm_eps) * w[-2]) @ w[-1].t()


def exact(case, seed):
    k = case["kind"]
    if k == "serve_tiny":
        weights = _tiny_weights(seed)
        reqs, forced = _tiny_requests(case, seed)
        out = []
        for r, f in zip(reqs, forced):
            logits = _tiny64(weights, np.concatenate([r.prompt, f]))
            out.append(logits[len(r.prompt) - 1:].numpy())
        return out
    if k == "gemm":
        x, w = _gemm_inputs(case, seed)
        return x.double() @ w.double().t()
    if k == "norm":
        x, part, gain = _norm_inputs(case, seed)
        x = x.double() + (part.double().sum(0) if part is not None else 0.0)
        return [x, _norm64(x, 1e-5) * gain.double()]
    if k == "decode_attn":
        ctx, q, kc, vc, bt = _decode_inputs(case, seed)
        rows = []
        for m, c in enumerate(ctx):
            kk, vv = _sequence(kc, vc, bt[m], c)
            rows.append(_attend64(q[m:m + 1], kk, vv, c - 1))
        return torch.cat(rows)
    if k == "prefill_attn":
        lens, q, kc, vc, bt = _prefill_inputs(case, seed)
        rows, at = [], 0
        for j, n in enumerate(lens):
            kk, vv = _sequence(kc, vc, bt[j], n)
            rows.append(_attend64(q[at:at + n], kk, vv, 0))
            at += n
        return torch.cat(rows)
    return None  # a service of random device weights; token ids
