"""Performance cases of the framework: the work a user has it do, each through
its public entry points (``paper_2604_07725_amd.sevo``).

Six kinds, at the decoder widths this repository names (the tiny test models,
the 8B- and 32B-class dense decoders, the 30B-A3B-class mixture of experts):

* ``step``   one decode step of a population (``StepBuffers.run``), a few layers
             of the decoder plus its LM head and the sampler;
* ``attn``   the paged decode attention of one layer (``sevo_attn_decode``);
* ``mlp``    norm, gate/up + SwiGLU and down projection of a layer, from one
             candidate to a prefill's thousands of tokens;
* ``sample`` the sampler on given logits (``sevo_logprob_sample``);
* ``pattn``  the causal attention of a prefill (``sevo_attn_prefill``), also
             of a trajectory continuing a cached prompt;
* ``score``  the confidence engine (``PrefillBuffers.run``): prompts and
             trajectories through a few layers, every scored row to its
             confidence, the keys and values appended to the cache.

Lengths follow from the case; every value follows from the seed.  ``exact``
computes the same in float64 with plain torch.
"""
import math

import torch

from paper_2604_07725_amd import sevo, synth

DEV = "cuda"
BF = torch.bfloat16

# decoder widths (hidden, q heads, kv heads, head dim, ffn, vocab, layers timed,
# experts, experts per token, expert ffn)
MODELS = {
    "tiny": (256, 4, 2, 64, 1024, 4096, 1, 0, 0, 0),
    "tiny_moe": (256, 4, 2, 64, 0, 4096, 2, 64, 4, 64),
    "dense8b": (4096, 32, 8, 128, 12288, 151936, 2, 0, 0, 0),
    "dense32b": (5120, 64, 8, 128, 25600, 151936, 2, 0, 0, 0),
    "moe30b": (2048, 32, 4, 128, 0, 151936, 2, 128, 8, 768),
}
HEADS = {"32/8": (32, 8, 128), "32/4": (32, 4, 128), "64/8": (64, 8, 128), "4/2": (4, 2, 64)}
CONF_K = 20
EPS = 1e-6
THETA = 1e6


def listed():
    return [
        # the test model's population of 4: every kernel is a launch and little else
        {"name": "step_tiny_n4", "kind": "step", "model": "tiny", "n": 4, "lo": 256, "hi": 512,
         "temp": 1.0, "top_k": 0, "top_p": 1.0},
        # a small population (4 candidates) of the 8B-class decoder on aggregation
        # prompts of a few thousand tokens: weights, read for four rows
        {"name": "step_dense8b_n4", "kind": "step", "model": "dense8b", "n": 4, "lo": 2048,
         "hi": 8192, "temp": 1.0, "top_k": 0, "top_p": 1.0},
        # the population of the throughput benchmark on the mixture of experts
        {"name": "step_moe30b_n64", "kind": "step", "model": "moe30b", "n": 64, "lo": 4096,
         "hi": 16384, "temp": 1.0, "top_k": 0, "top_p": 1.0},
        # decode attention of 16 candidates, four aggregated answers each
        {"name": "attn_n16", "kind": "attn", "heads": "32/8", "n": 16, "lo": 8192, "hi": 16384},
        # decode attention of the benchmark's 64 candidates at 16k-32k tokens: the
        # step's largest part
        {"name": "attn_n64", "kind": "attn", "heads": "32/8", "n": 64, "lo": 16384, "hi": 32768},
        # the FFN of a decode step for a population of 128 (circle packing)
        {"name": "mlp_n128", "kind": "mlp", "model": "dense8b", "m": 128},
        # the FFN of a prefill chunk
        {"name": "mlp_t8192", "kind": "mlp", "model": "dense8b", "m": 8192},
        # the sampler at the top-k / top-p row of the generation hyper-parameters
        {"name": "sample_topk_n16", "kind": "sample", "n": 16, "vocab": 151936, "temp": 0.7,
         "top_k": 20, "top_p": 0.8, "min_p": 0.0, "conf": CONF_K},
        # prefill attention of one long request (the confidence benchmark's 40K)
        {"name": "pattn_40k", "kind": "pattn", "heads": "32/8", "seqs": 1, "lo": 40960,
         "hi": 40960, "prefix": 0},
        # trajectories of different lengths behind cached prompts, scored together
        {"name": "pattn_ragged", "kind": "pattn", "heads": "32/8", "seqs": 6, "lo": 300,
         "hi": 3000, "prefix": 2000},
        # cross-model confidence of a few short answers, half of each prompt
        {"name": "score_dense8b", "kind": "score", "model": "dense8b", "seqs": 3, "lo": 400,
         "hi": 1100, "scored": 0.5},
        # the same on the mixture of experts, two longer ones
        {"name": "score_moe30b", "kind": "score", "model": "moe30b", "seqs": 2, "lo": 3000,
         "hi": 5000, "scored": 0.25},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "attn", "mlp", "mlp", "sample", "pattn", "score"])
    if kind == "step":
        model = rng.choice(["tiny", "tiny_moe", "dense8b", "dense32b", "moe30b"])
        n = _log_int(rng, 1, 128)
        hi = min(_log_int(rng, 256, 32768), max(256, 1_000_000 // n))
        top_k = rng.choice([0, 20])
        return {"kind": kind, "model": model, "n": n, "lo": max(16, int(hi * rng.uniform(0.3, 1.0))),
                "hi": hi, "temp": rng.choice([0.0, 0.6, 1.0]), "top_k": top_k,
                "top_p": rng.choice([0.8, 0.95]) if top_k else 1.0}
    if kind == "attn":
        n = _log_int(rng, 1, 128)
        hi = min(_log_int(rng, 256, 65536), max(256, 1_500_000 // n))
        return {"kind": kind, "heads": rng.choice(sorted(HEADS)), "n": n,
                "lo": max(1, int(hi * rng.uniform(0.1, 1.0))), "hi": hi}
    if kind == "mlp":
        return {"kind": kind, "model": rng.choice(["dense8b", "dense8b", "dense32b"]),
                "m": _log_int(rng, 1, 8192)}
    if kind == "sample":
        top_k = rng.choice([0, 10, 20, 32])
        return {"kind": kind, "n": _log_int(rng, 1, 256), "vocab": rng.choice([4096, 32000, 151936]),
                "temp": rng.choice([0.0, 0.7, 1.0]), "top_k": top_k,
                "top_p": rng.choice([0.8, 0.95, 1.0]) if top_k else 1.0,
                "min_p": rng.choice([0.0, 0.05]) if top_k else 0.0, "conf": rng.choice([0, CONF_K])}
    if kind == "pattn":
        seqs = rng.choice([1, 1, 2, 4, 8])
        hi = _log_int(rng, 64, 24576 // seqs)
        return {"kind": kind, "heads": rng.choice(sorted(HEADS)), "seqs": seqs,
                "lo": max(1, int(hi * rng.uniform(0.1, 1.0))), "hi": hi,
                "prefix": rng.choice([0, 0, _log_int(rng, 16, 4096)])}
    seqs = rng.choice([1, 2, 4])
    hi = _log_int(rng, 128, 8192 // seqs)
    return {"kind": kind, "model": rng.choice(["tiny", "tiny_moe", "dense8b", "moe30b"]), "seqs": seqs,
            "lo": max(8, int(hi * rng.uniform(0.3, 1.0))), "hi": hi,
            "scored": rng.choice([0.1, 0.25, 0.5])}


# ------------------------------------------------------------------ inputs
def _gen(seed, what):
    return torch.Generator(device=DEV).manual_seed(int(seed) * 1000 + what)


def _normal(shape, std, g, mean=0.0, dtype=BF):
    return torch.empty(shape, dtype=dtype, device=DEV).normal_(mean, std, generator=g)


def _lens(n, lo, hi):
    """n lengths spread over [lo, hi] (a fixed low-discrepancy order)."""
    return [lo + int(round((hi - lo) * ((i + 1) * 0.6180339887498949 % 1.0))) for i in range(n)]


def _shape(name):
    hidden, hq, hkv, d, ffn, vocab, layers, E, k, fe = MODELS[name]
    return synth.ModelShape(layers, hidden, hq, hkv, d, ffn, vocab, rope_theta=THETA, rms_eps=EPS,
                            n_experts=E, top_k=k, expert_ffn=fe)


def _plain_weights(name, seed):
    """The decoder's weights, row-major [out][in]."""
    s, g = _shape(name), _gen(seed, 1)
    H = s.hidden

    def w(*shape):
        return _normal(shape, 0.02, g)

    def gain(n):
        return _normal((n,), 0.02, g, mean=1.0)

    # the residual stream of a trained decoder is large next to one layer's update
    out = {"embed": _normal((s.vocab, H), 1.0, g), "lm_head": w(s.vocab, H),
           "final_norm": gain(H), "layers": []}
    for _ in range(s.n_layers):
        t = {"attn_norm": gain(H), "w_qkv": w(s.qkv_dim, H), "q_norm": gain(s.head_dim),
             "k_norm": gain(s.head_dim), "w_o": w(H, s.q_dim), "ffn_norm": gain(H)}
        if s.is_moe:
            t["w_router"] = w(s.n_experts, H)
            t["w_expert_gate_up"] = w(s.n_experts, 2 * s.expert_ffn, H)
            t["w_expert_down"] = w(s.n_experts, H, s.expert_ffn)
        else:
            t["w_gate_up"] = w(2 * s.ffn, H)
            t["w_down"] = w(H, s.ffn)
        out["layers"].append(t)
    return out


def _pack(name, t):
    if name not in sevo.PACKED_WEIGHTS:
        return t
    kind = sevo.PACKED_WEIGHTS[name]
    if t.dim() == 2:
        return sevo.sevo_pack_weight(t, kind)
    out = torch.empty_like(t)
    for e in range(t.shape[0]):
        sevo.sevo_pack_weight(t[e], kind, dst=out[e])
    return out


def _model(name, seed, max_position):
    plain = _plain_weights(name, seed)
    packed = {k: _pack(k, v) for k, v in plain.items() if k != "layers"}
    packed["layers"] = [{k: _pack(k, v) for k, v in t.items()} for t in plain["layers"]]
    return sevo.sevo_init_model(_shape(name), packed, max_position)


def _pages(lens, seed):
    """Page table int32 [n][max_pages] (random physical pages, -1 past the end)
    holding lens[i] tokens each, and the pool's page count."""
    need = [(t + 15) // 16 for t in lens]
    total, width = sum(need), max(need)
    perm = torch.randperm(total, generator=_gen(seed, 2), device=DEV).to(torch.int32)
    pt = torch.full((len(lens), width), -1, dtype=torch.int32, device=DEV)
    at = 0
    for i, k in enumerate(need):
        pt[i, :k] = perm[at:at + k]
        at += k
    return pt, total


def _plain_kv(pages, hkv, d, seed, layer=0):
    g = _gen(seed, 100 + layer)
    return _normal((pages, hkv, 16, d), 1.0, g), _normal((pages, hkv, 16, d), 1.0, g)


def _ints(n, high, seed, what, dtype=torch.int32):
    return torch.randint(0, high, (n,), generator=_gen(seed, what), device=DEV, dtype=dtype)


def _starts(lens):
    s = [0]
    for t in lens:
        s.append(s[-1] + t)
    return torch.tensor(s, dtype=torch.int32, device=DEV)


def _prefixes(case):
    """Cached tokens before each sequence (0 without a prefix)."""
    p = case["prefix"]
    return [0] * case["seqs"] if not p else _lens(case["seqs"], p // 4, p)


def _scored_rows(case):
    """The last share of every sequence's rows, as packed token indices."""
    rows, at = [], 0
    for t in _lens(case["seqs"], case["lo"], case["hi"]):
        k = max(1, int(t * case["scored"]))
        rows += range(at + t - k, at + t)
        at += t
    return rows


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        lens = _lens(case["n"], case["lo"], case["hi"])
        s = _shape(case["model"])
        model = _model(case["model"], seed, max(lens) + 1)
        pt, pages = _pages([t + 1 for t in lens], seed)
        pools = [sevo.sevo_pack_kv(*_plain_kv(pages, s.n_kv_heads, s.head_dim, seed, l))
                 for l in range(s.n_layers)]
        pos = torch.tensor(lens, dtype=torch.int32, device=DEV)
        buf = sevo.StepBuffers(model, _ints(case["n"], s.vocab, seed, 3), pos, pt, pools,
                               _ints(case["n"], 1 << 62, seed, 4, torch.int64), seed=seed,
                               temperature=case["temp"], keep_logits=True, conf_topk=CONF_K,
                               top_k=case["top_k"], top_p=case["top_p"])
        return {"case": case, "buf": buf, "pools": pools}
    if kind == "attn":
        hq, hkv, d = HEADS[case["heads"]]
        lens = _lens(case["n"], case["lo"], case["hi"])
        pt, pages = _pages(lens, seed)
        pool = sevo.sevo_pack_kv(*_plain_kv(pages, hkv, d, seed))
        q = _normal((case["n"], hq, d), 1.0, _gen(seed, 5))
        need = sevo.sevo_attn_workspace_bytes(case["n"], hq, hkv, d, pt.shape[1])
        return {"case": case, "q": q, "pool": pool, "pt": pt, "out": torch.empty_like(q),
                "lens": torch.tensor(lens, dtype=torch.int32, device=DEV),
                "ws": torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)}
    if kind == "mlp":
        x, gain, wgu, wd = _mlp_inputs(case, seed)
        m, H, F = case["m"], wd.shape[0], wd.shape[1]
        m16 = -(-m // 16) * 16
        need = max(sevo.sevo_linear_workspace_bytes(m, H, F), 256)
        return {"case": case, "x": x, "gain": gain,
                "wgu": sevo.sevo_pack_weight(wgu, sevo.PACK_GATE_UP),
                "wd": sevo.sevo_pack_weight(wd),
                "h": torch.zeros(m16 * H, dtype=BF, device=DEV),
                "a": torch.zeros(m16, F, dtype=BF, device=DEV),
                "y": torch.empty(m, H, dtype=torch.float32, device=DEV),
                "ws": torch.empty(need, dtype=torch.uint8, device=DEV)}
    if kind == "sample":
        logits, uid, pos = _sample_inputs(case, seed)
        n = case["n"]
        need = sevo.sevo_sample_workspace_bytes(n, case["vocab"])
        return {"case": case, "logits": logits, "uid": uid, "pos": pos, "seed": seed,
                "ids": torch.empty(n, dtype=torch.int32, device=DEV),
                "lps": torch.empty(n, dtype=torch.float32, device=DEV),
                "conf": torch.empty(n, dtype=torch.float32, device=DEV) if case["conf"] else None,
                "ws": torch.empty(max(need, 256), dtype=torch.uint8, device=DEV)}
    if kind == "pattn":
        hq, hkv, d = HEADS[case["heads"]]
        lens = _lens(case["seqs"], case["lo"], case["hi"])
        pre = _prefixes(case)
        pt, pages = _pages([t + p for t, p in zip(lens, pre)], seed)
        q = _normal((sum(lens), hq, d), 1.0, _gen(seed, 5))
        return {"case": case, "q": q, "pool": sevo.sevo_pack_kv(*_plain_kv(pages, hkv, d, seed)),
                "pt": pt, "starts": _starts(lens), "max": max(lens), "out": torch.empty_like(q),
                "start_pos": (torch.tensor(pre, dtype=torch.int32, device=DEV)
                              if case["prefix"] else None)}
    lens = _lens(case["seqs"], case["lo"], case["hi"])
    s = _shape(case["model"])
    model = _model(case["model"], seed, max(lens))
    pt, pages = _pages(lens, seed)
    pools = [sevo.sevo_pack_kv(*_plain_kv(pages, s.n_kv_heads, s.head_dim, seed, l))
             for l in range(s.n_layers)]
    rows = torch.tensor(_scored_rows(case), dtype=torch.int32, device=DEV)
    buf = sevo.PrefillBuffers(model, _ints(sum(lens), s.vocab, seed, 3), _starts(lens), pt, pools,
                              rows, CONF_K, max(lens))
    return {"case": case, "buf": buf, "pools": pools}


def _mlp_inputs(case, seed):
    s, g = _shape(case["model"]), _gen(seed, 6)
    x = _normal((case["m"], s.hidden), 1.0, g, dtype=torch.float32)
    gain = _normal((s.hidden,), 0.02, g, mean=1.0)
    return x, gain, _normal((2 * s.ffn, s.hidden), 0.02, g), _normal((s.hidden, s.ffn), 0.02, g)


def _sample_inputs(case, seed):
    logits = _normal((case["n"], case["vocab"]), 2.0, _gen(seed, 7), dtype=torch.float32)
    return (logits, _ints(case["n"], 1 << 62, seed, 4, torch.int64),
            _ints(case["n"], 65536, seed, 8))


# ------------------------------------------------------------------ the pass
def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        # the token ids are an arg-max over these logits, which a last-bit
        # difference can turn: the sampler's own cases compare them
        b = state["buf"]
        _, lps = b.run()
        return {"logits": b.out_logits, "lps": lps, "conf": b.out_conf, "pools": state["pools"]}
    if kind == "attn":
        return sevo.sevo_attn_decode(state["q"], state["pool"], state["pt"], state["lens"],
                                     out=state["out"], workspace=state["ws"])
    if kind == "mlp":
        m = case["m"]
        sevo.sevo_add_rmsnorm(state["x"], None, state["gain"], EPS, out=state["h"])
        sevo.sevo_linear(state["h"], state["wgu"], sevo.LINEAR_SWIGLU, out=state["a"], m=m,
                         x_tiled=True, out_tiled=True, workspace=state["ws"])
        return sevo.sevo_linear(state["a"], state["wd"], sevo.LINEAR_STORE, out=state["y"], m=m,
                                x_tiled=True, workspace=state["ws"])
    if kind == "sample":
        out = sevo.sevo_logprob_sample(
            state["logits"], case["temp"], state["seed"], state["uid"], state["pos"],
            out_tokens=state["ids"], out_logprobs=state["lps"], workspace=state["ws"],
            conf_topk=case["conf"], out_conf=state["conf"], top_k=case["top_k"],
            top_p=case["top_p"], min_p=case["min_p"])
        return dict(zip(("ids", "lps", "conf"), out))
    if kind == "pattn":
        return sevo.sevo_attn_prefill(state["q"], state["pool"], state["pt"], state["starts"],
                                      state["max"], start_pos=state["start_pos"],
                                      out=state["out"])
    b = state["buf"]
    return {"conf": b.run(), "rows": b.out_row_conf, "pools": state["pools"]}


# ------------------------------------------------------------------ what a pass cannot do without
def _decoder_work(s, tokens, logit_rows):
    """(weight bytes read once, projection flops) of `tokens` through the decoder."""
    H = s.hidden
    attn = s.qkv_dim * H + H * s.q_dim
    if s.is_moe:
        # experts touched under uniform routing
        hit = s.n_experts * (1.0 - (1.0 - s.top_k / s.n_experts) ** tokens)
        per = 3 * s.expert_ffn * H
        read = attn + s.n_experts * H + hit * per
        done = attn + s.n_experts * H + s.top_k * per
    else:
        read = done = attn + 3 * s.ffn * H
    return (2.0 * (s.n_layers * read + s.vocab * H),
            2.0 * (s.n_layers * done * tokens + s.vocab * H * logit_rows))


def work(case):
    kind = case["kind"]
    if kind == "step":
        s = _shape(case["model"])
        n, lens = case["n"], _lens(case["n"], case["lo"], case["hi"])
        wb, wf = _decoder_work(s, n, n)
        keys = sum(lens) + n
        return {"bytes": wb + s.n_layers * (4.0 * s.kv_dim * keys) + n * (2.0 * s.hidden + 4.0 * s.vocab),
                "flops": wf + s.n_layers * 4.0 * s.q_dim * keys}
    if kind == "attn":
        hq, hkv, d = HEADS[case["heads"]]
        keys = sum(_lens(case["n"], case["lo"], case["hi"]))
        return {"bytes": 4.0 * hkv * d * keys + 4.0 * case["n"] * hq * d + keys / 4.0,
                "flops": 4.0 * hq * d * keys}
    if kind == "mlp":
        s, m = _shape(case["model"]), case["m"]
        return {"bytes": 6.0 * s.ffn * s.hidden + 8.0 * m * s.hidden, "flops": 6.0 * m * s.ffn * s.hidden}
    if kind == "sample":
        return {"bytes": 4.0 * case["n"] * case["vocab"], "flops": 0.0}
    lens = _lens(case["seqs"], case["lo"], case["hi"])
    pairs = sum(t * (t + 1) / 2 for t in lens)
    if kind == "pattn":
        hq, hkv, d = HEADS[case["heads"]]
        pre = _prefixes(case)
        pairs += sum(t * p for t, p in zip(lens, pre))
        return {"bytes": 4.0 * sum(lens) * hq * d + 4.0 * hkv * d * (sum(lens) + sum(pre)),
                "flops": 4.0 * hq * d * pairs}
    s = _shape(case["model"])
    wb, wf = _decoder_work(s, sum(lens), len(_scored_rows(case)))
    return {"bytes": wb + sum(lens) * (2.0 * s.hidden + s.n_layers * 4.0 * s.kv_dim),
            "flops": wf + s.n_layers * 4.0 * s.q_dim * pairs}


def tolerance(case):
    # about four times the difference of two correct orders of the sums; bf16
    # storage points turn a last bit into a bf16 step now and then
    return {
        # logits after a few layers; a near tie may sample another token, whose
        # log-probability then differs
        "step": {"rel": 0.02, "max": 0.6},
        # outputs rounded to bf16
        "attn": {"rel": 3e-3, "max": 0.05},
        # one bf16 product between two fp32 sums
        "mlp": {"rel": 2e-3, "max": 0.02},
        "sample": {"rel": 1e-5, "max": 1e-3, "differ": 0.01},
        # probabilities rounded to bf16
        "pattn": {"rel": 8e-3, "max": 0.2},
        # confidences after a few layers, keys and values in bf16
        "score": {"rel": 8e-3, "max": 0.6},
    }[case["kind"]]


# ------------------------------------------------------------------ the same in float64
def _rms(x, gain):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.double()


def _lin(x, w):
    """x w^T in float64, a slab of rows of w at a time."""
    if w.numel() <= 1 << 28:
        return x @ w.double().t()
    step = max(1, (1 << 28) // w.shape[1])
    return torch.cat([x @ w[i:i + step].double().t() for i in range(0, w.shape[0], step)], 1)


def _rope(x, pos):
    half = x.shape[-1] // 2
    inv = THETA ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / x.shape[-1])
    ang = pos.double()[:, None, None] * inv
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], -1)


def _swiglu(gu):
    g, u = gu.chunk(2, -1)
    return g * torch.sigmoid(g) * u


def _keys(pool, pt_row, n):
    """Logical rows 0..n-1 of a plain pool, float64 [hkv][n][d]."""
    p = pool[pt_row[:(n + 15) // 16].long()]
    return p.transpose(0, 1).reshape(pool.shape[1], -1, pool.shape[3])[:, :n].double()


def _attend(q, k, v, first):
    """Causal attention of q [t][hq][d] at positions first.. over k, v [hkv][n][d]."""
    t, hq, d = q.shape
    hkv, n = k.shape[:2]
    g = hq // hkv
    out = torch.empty_like(q)
    block = 1024
    for c in range(hkv):
        for t0 in range(0, t, block):
            t1 = min(t, t0 + block)
            m = min(n, first + t1)
            qq = q[t0:t1, c * g:(c + 1) * g].reshape(-1, d)
            s = (qq @ k[c, :m].t()) * d ** -0.5
            at = torch.arange(first + t0, first + t1, device=DEV).repeat_interleave(g)
            s.masked_fill_(torch.arange(m, device=DEV)[None, :] > at[:, None], -math.inf)
            out[t0:t1, c * g:(c + 1) * g] = (torch.softmax(s, -1) @ v[c, :m]).reshape(t1 - t0, g, d)
    return out


def _moe(h, t, s):
    top, idx = torch.topk(_lin(h, t["w_router"]), s.top_k, dim=-1)
    wt = torch.softmax(top, -1)
    y = torch.zeros_like(h)
    for e in range(s.n_experts):
        tok, slot = (idx == e).nonzero(as_tuple=True)
        if tok.numel():
            a = _swiglu(_lin(h[tok], t["w_expert_gate_up"][e]))
            y.index_add_(0, tok, _lin(a, t["w_expert_down"][e]) * wt[tok, slot][:, None])
    return y


def _fused(k, v):
    """Plain K, V [pages][hkv][16][d] -> the fused pool's element order."""
    p, h, _, d = k.shape
    kt = k.reshape(p, h, 16, d // 32, 32).transpose(2, 3).reshape(p, h, 16 * d)
    return torch.stack([kt, v.transpose(2, 3).reshape(p, h, 16 * d)], 2)


def _decoder(case, seed, lens, pre, tokens):
    """(final residual stream, updated pools, weights): `lens` new tokens per
    sequence behind `pre` cached ones."""
    s, w = _shape(case["model"]), _plain_weights(case["model"], seed)
    pt, pages = _pages([t + p for t, p in zip(lens, pre)], seed)
    pos = torch.cat([torch.arange(p, p + t, device=DEV) for t, p in zip(lens, pre)])
    row = torch.cat([torch.full((t,), i, device=DEV) for i, t in enumerate(lens)])
    page, slot = pt[row, pos // 16].long(), pos % 16
    x = w["embed"][tokens.long()].double()
    pools = []
    for l, t in enumerate(w["layers"]):
        k_pool, v_pool = _plain_kv(pages, s.n_kv_heads, s.head_dim, seed, l)
        h = _rms(x, t["attn_norm"])
        qkv = _lin(h, t["w_qkv"]).reshape(len(row), -1, s.head_dim)
        q, k, v = qkv.split([s.n_q_heads, s.n_kv_heads, s.n_kv_heads], 1)
        q, k = _rope(_rms(q, t["q_norm"]), pos), _rope(_rms(k, t["k_norm"]), pos)
        o, at = torch.empty_like(q), 0
        for i, (n, p) in enumerate(zip(lens, pre)):
            kk = torch.cat([_keys(k_pool, pt[i], p), k[at:at + n].transpose(0, 1)], 1)
            vv = torch.cat([_keys(v_pool, pt[i], p), v[at:at + n].transpose(0, 1)], 1)
            o[at:at + n] = _attend(q[at:at + n], kk, vv, p)
            at += n
        k64, v64 = k_pool.double(), v_pool.double()
        k64[page, :, slot], v64[page, :, slot] = k, v
        pools.append(_fused(k64, v64))
        x = x + _lin(o.reshape(len(row), -1), t["w_o"])
        h = _rms(x, t["ffn_norm"])
        x = x + (_moe(h, t, s) if s.is_moe else _lin(_swiglu(_lin(h, t["w_gate_up"])), t["w_down"]))
    return x, pools, w


def _confidence(logits):
    return torch.logsumexp(logits, -1) - torch.topk(logits, CONF_K, dim=-1).values.mean(-1)


def _mul_hi_lo(a, b):
    """High and low 32 bits of a product of 32-bit values held in int64."""
    ah, al, bh, bl = a >> 16, a & 0xFFFF, b >> 16, b & 0xFFFF
    lo = al * bl
    mid = ah * bl + (lo >> 16)
    mid2 = al * bh + (mid & 0xFFFF)
    return (ah * bh + (mid >> 16) + (mid2 >> 16)) & 0xFFFFFFFF, ((mid2 & 0xFFFF) << 16) | (lo & 0xFFFF)


def _gumbel(uid, pos, vocab, seed):
    """The sampler's noise (Philox4x32-10 keyed by candidate and position), float64 [vocab]."""
    c0 = torch.arange((vocab + 3) // 4, device=DEV)
    c1, c2, c3 = (torch.full_like(c0, v) for v in (pos, uid & 0xFFFFFFFF, uid >> 32))
    k0, k1 = seed & 0xFFFFFFFF, seed >> 32
    for _ in range(10):
        h0, l0 = _mul_hi_lo(c0, 0xD2511F53)
        h1, l1 = _mul_hi_lo(c2, 0xCD9E8D57)
        c0, c1, c2, c3 = h1 ^ c1 ^ k0, l1, h0 ^ c3 ^ k1, l0
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    u = ((torch.stack([c0, c1, c2, c3], 1).reshape(-1)[:vocab] >> 9).double() + 0.5) * 2.0 ** -23
    return -torch.log(-torch.log(u))


def _exact_sample(case, seed):
    logits, uid, pos = _sample_inputs(case, seed)
    T = case["temp"]
    ids, lps, conf = [], [], []
    for i in range(case["n"]):
        x = logits[i].double()
        z = x / T if T else x
        if case["top_k"]:
            v, order = torch.topk(x, case["top_k"])
            zz = v / T if T else v
            keep = torch.ones_like(zz, dtype=torch.bool)
            if case["min_p"] > 0:
                keep &= zz >= zz[0] + math.log(case["min_p"])
            p = torch.exp(zz - zz[0]) * keep
            before = torch.cumsum(p, 0) - p
            keep &= before < case["top_p"] * p.sum() if case["top_p"] < 1 else keep
            kept = torch.full_like(x, -math.inf)
            kept[order[keep]] = z[order[keep]]
            z = kept
        g = _gumbel(int(uid[i]), int(pos[i]), case["vocab"], seed) if T else 0.0
        k = int(torch.argmax(z + g))
        ids.append(k)
        lps.append(z[k] - torch.logsumexp(z, 0))
        conf.append(_confidence(x))
    out = {"ids": torch.tensor(ids, dtype=torch.int32), "lps": torch.stack(lps)}
    return dict(out, conf=torch.stack(conf)) if case["conf"] else out


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        lens = _lens(case["n"], case["lo"], case["hi"])
        tokens = _ints(case["n"], _shape(case["model"]).vocab, seed, 3)
        x, pools, w = _decoder(case, seed, [1] * case["n"], lens, tokens)
        logits = _lin(_rms(x, w["final_norm"]), w["lm_head"])
        return {"logits": logits, "lps": None, "conf": _confidence(logits), "pools": pools}
    if kind == "attn":
        hq, hkv, d = HEADS[case["heads"]]
        lens = _lens(case["n"], case["lo"], case["hi"])
        pt, pages = _pages(lens, seed)
        k, v = _plain_kv(pages, hkv, d, seed)
        q = _normal((case["n"], hq, d), 1.0, _gen(seed, 5)).double()
        return torch.cat([_attend(q[i:i + 1], _keys(k, pt[i], t), _keys(v, pt[i], t), t - 1)
                          for i, t in enumerate(lens)])
    if kind == "mlp":
        x, gain, wgu, wd = _mlp_inputs(case, seed)
        return torch.cat([_lin(_swiglu(_lin(_rms(c.double(), gain), wgu)), wd)
                          for c in x.split(4096)])
    if kind == "sample":
        return _exact_sample(case, seed)
    lens = _lens(case["seqs"], case["lo"], case["hi"])
    if kind == "pattn":
        hq, hkv, d = HEADS[case["heads"]]
        pre = _prefixes(case)
        pt, pages = _pages([t + p for t, p in zip(lens, pre)], seed)
        k, v = _plain_kv(pages, hkv, d, seed)
        q = _normal((sum(lens), hq, d), 1.0, _gen(seed, 5)).double()
        out = []
        for i, (part, p) in enumerate(zip(q.split(lens), pre)):
            n = p + len(part)
            out.append(_attend(part, _keys(k, pt[i], n), _keys(v, pt[i], n), p))
        return torch.cat(out)
    tokens = _ints(sum(lens), _shape(case["model"]).vocab, seed, 3)
    x, pools, w = _decoder(case, seed, lens, [0] * len(lens), tokens)
    rows = torch.tensor(_scored_rows(case), device=DEV)
    c = torch.cat([_confidence(_lin(_rms(x[r], w["final_norm"]), w["lm_head"]))
                   for r in rows.split(1024)])
    starts = _starts(lens).tolist()
    mean = [c[(rows >= a) & (rows < b)].mean() for a, b in zip(starts, starts[1:])]
    return {"conf": torch.stack(mean), "rows": c, "pools": pools}
