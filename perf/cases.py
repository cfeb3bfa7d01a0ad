"""The work that users of this framework have it do, as cases that can be timed and compared.

A case is a dict of plain values.  Five kinds, each through the public calls of
paper_2606_03113_amd (the C ABI's names):

  prefill   lede_prefill of `n` tokens behind `ctx` cached ones: a first prompt, or a further turn
  decode    a generation of `n` tokens from a cached context by one of the four kinds of step:
            "ssd" (forced exit layer and draft length, the Q-network logged), "ar" (no drafts),
            "sampled" (speculative sampling) and "policy" (the exit policy decides)
  linear    lede_op_linear: one projection of a verify pass
  sample    lede_op_sample_noalloc: draws from logits rows, as a serving loop takes them
  update    lede_dqn_update: one learning update of the exit policy's trainer

Models have the widths of the repository's workloads and mostly a few of their layers, so that a
case is a block of layers with a tolerance of its own.  Their weights are random with unit-variance
projections, residual projections scaled down by the depth, and a head that knows each token's
successor: like a trained model, and unlike a plain random one, the next token has a clear margin,
early exits agree with the full model and drafts are accepted.
"""
import ctypes
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2606_03113_amd import lede

# d_model, heads, KV heads, head dim, ffn, vocabulary, dtype, rotary base: the repository's workloads
SHAPES = {
    "tiny": (256, 4, 4, 64, 688, 1024, "f32", 10000.0),
    "llama2-7b": (4096, 32, 32, 128, 11008, 32000, "bf16", 10000.0),
    "llama3-8b": (4096, 32, 8, 128, 14336, 128256, "bf16", 500000.0),
    "llama2-13b": (5120, 40, 40, 128, 13824, 32000, "bf16", 10000.0),
    "llama2-70b": (8192, 64, 8, 128, 28672, 32000, "bf16", 10000.0),
}
EPS = 1e-5
MARGIN = 18.0        # the successor's logit before the layers' noise
TEMPERATURE = 0.6
POLICY_HIDDEN = 16
PREFILL_LIMIT = 4096 * 2 * 317e6  # tokens x layer parameters of the largest listed prefill


def listed():
    return [
        # the smallest call: one learning update with the paper's hyperparameters
        {"name": "update", "kind": "update", "hidden": 16, "batch": 32, "n_step": 3},
        # draws for the five rows of a verify pass
        {"name": "sample", "kind": "sample", "rows": 5, "vocab": 32000},
        # the down projection of a verify of eight drafts
        {"name": "linear", "kind": "linear", "n_out": 5120, "n_in": 13824, "rows": 9},
        # the smallest model (fp32): a whole generation, all latency and launches
        {"name": "tiny", "kind": "decode", "shape": "tiny", "layers": 4, "mode": "ssd", "ctx": 32, "n": 64, "l": 2, "k": 4},
        # a further turn of a conversation: a short prompt of odd length behind a cached one, grouped heads
        {"name": "turn", "kind": "prefill", "shape": "llama3-8b", "layers": 2, "ctx": 1024, "n": 97},
        # the ordinary prompt
        {"name": "prompt", "kind": "prefill", "shape": "llama2-7b", "layers": 4, "ctx": 0, "n": 512},
        # the longest prompt
        {"name": "document", "kind": "prefill", "shape": "llama2-13b", "layers": 2, "ctx": 0, "n": 4096},
        # the whole model: self-speculative decoding at the headline exit layer and draft length
        {"name": "ssd", "kind": "decode", "shape": "llama2-7b", "layers": 32, "mode": "ssd", "ctx": 512, "n": 15, "l": 8, "k": 4},
        # plain autoregressive decoding, the widest layers
        {"name": "ar", "kind": "decode", "shape": "llama2-70b", "layers": 2, "mode": "ar", "ctx": 2048, "n": 4, "l": 1, "k": 0},
        # long context, eight drafts
        {"name": "long", "kind": "decode", "shape": "llama2-13b", "layers": 4, "mode": "ssd", "ctx": 4096, "n": 18, "l": 2, "k": 8},
        # speculative sampling, the largest vocabulary
        {"name": "sampled", "kind": "decode", "shape": "llama3-8b", "layers": 4, "mode": "sampled", "ctx": 1024, "n": 14, "l": 2, "k": 6},
        # the exit policy: a decision per draft, twelve drafts
        {"name": "policy", "kind": "decode", "shape": "llama2-7b", "layers": 8, "mode": "policy", "ctx": 520, "n": 13, "l": 2, "k": 12},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49))))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "decode", "decode", "decode", "linear", "sample", "update"])
    if kind == "update":
        hidden = _log_int(rng, 4, 128)
        return {"kind": kind, "hidden": hidden, "batch": _log_int(rng, 4, min(256, 4096 // hidden)), "n_step": rng.randint(1, 5)}
    if kind == "sample":
        return {"kind": kind, "rows": rng.randint(1, 16), "vocab": _log_int(rng, 1000, 128256)}
    if kind == "linear":
        return {"kind": kind, "n_out": 16 * _log_int(rng, 64, 1792), "n_in": _log_int(rng, 1024, 28672), "rows": rng.randint(1, 16)}
    shape = rng.choice(list(SHAPES))
    layers = 4 if shape == "tiny" else rng.randint(1, 4)
    if kind == "prefill":
        most = 4096 if shape != "tiny" else 512
        most = min(most, int(PREFILL_LIMIT / (layers * _layer_params(_model({"shape": shape, "layers": layers})))))
        return {"kind": kind, "shape": shape, "layers": layers, "ctx": rng.choice([0, 0, _log_int(rng, 16, 2048)]), "n": _log_int(rng, 8, most)}
    mode = rng.choice(["ssd", "ssd", "ar", "sampled", "policy"])
    k = 0 if mode == "ar" else 12 if mode == "policy" else rng.randint(1, 12)
    return {"kind": kind, "shape": shape, "layers": layers, "mode": mode, "ctx": _log_int(rng, 32, 4096 if shape != "tiny" else 512),
            "n": rng.randint(2, 13) if mode == "ar" else rng.randint(max(2, k // 2), 2 * k + 4), "l": rng.randint(1, layers), "k": k}


# ---- models and inputs ---------------------------------------------------------------------


def _model(case):
    d, nq, nkv, hd, ffn, vocab, dtype, base = SHAPES[case["shape"]]
    first = case.get("l", 1) if case.get("mode") == "policy" else 1
    return SimpleNamespace(n_layers=case["layers"], d_model=d, n_heads=nq, n_kv_heads=nkv, head_dim=hd, ffn_dim=ffn, vocab=vocab,
                           dtype=dtype, rope_base=base, rms_eps=EPS, qnet_hidden=256 if d > 256 else 64,
                           exits=tuple(range(first, case["layers"] + 1)), lengths=(2, 4, 6, 8))


def _layer_params(m):
    return m.d_model * (2 * m.n_heads + 2 * m.n_kv_heads) * m.head_dim + 3 * m.d_model * m.ffn_dim


def _generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def _weights(m, g):
    """Device tensors in lede_load_weights' layout, and each token's successor."""
    dt = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    d, qd, kvd, f, V, L = m.d_model, m.n_heads * m.head_dim, m.n_kv_heads * m.head_dim, m.ffn_dim, m.vocab, m.n_layers

    def normal(*shape, std):
        return torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, std, generator=g)

    def gain():
        return torch.empty(d, dtype=dt, device="cuda").normal_(1.0, 0.1, generator=g)

    succ = torch.randperm(V, device="cuda", generator=g)
    embed = normal(V, d, std=1.0)
    head = normal(V, d, std=d ** -0.5)
    head[succ] += embed * (MARGIN / d)
    w = {"embed": embed, "head": head, "final_norm": gain(), "layers": []}
    for _ in range(L):
        w["layers"].append({
            "attn_norm": gain(), "wq": normal(qd, d, std=1.28 * d ** -0.5), "wk": normal(kvd, d, std=1.28 * d ** -0.5),
            "wv": normal(kvd, d, std=1.28 * d ** -0.5), "wo": normal(d, qd, std=(2 * L * qd) ** -0.5), "ffn_norm": gain(),
            "wg": normal(f, d, std=1.28 * d ** -0.5), "wu": normal(f, d, std=1.28 * d ** -0.5),
            "wd": normal(d, f, std=(2 * L * f) ** -0.5)})
    return w, succ


def _qnets(m, seed):
    """The (exit, length) Q-network, and an exit-policy network that exits when the top tokens stand out."""
    r = np.random.default_rng(seed)
    H, A, He = m.qnet_hidden, len(m.exits) * len(m.lengths), POLICY_HIDDEN
    q = {"w1": (r.standard_normal((H, m.d_model)) * m.d_model ** -0.5).astype(np.float32), "b1": (0.1 * r.standard_normal(H)).astype(np.float32),
         "w2": (r.standard_normal((A, H)) * H ** -0.5).astype(np.float32), "b2": (0.1 * r.standard_normal(A)).astype(np.float32)}
    e = {"w1": (0.05 * r.standard_normal((He, 3))).astype(np.float32), "b1": (0.05 * r.standard_normal(He)).astype(np.float32),
         "w2": (0.05 * r.standard_normal((2, He))).astype(np.float32), "b2": np.zeros(2, np.float32)}
    e["w1"][0], e["b1"][0], e["w2"][:, 0] = (1.0, 0.0, 0.0), -2.0, (0.0, 1.0)
    return q, e


def _tokens(case, m, g):
    ctx = case["ctx"] if case["kind"] == "decode" else case["ctx"] + case["n"]
    return torch.randint(0, m.vocab, (ctx,), device="cuda", generator=g).cpu().numpy().astype(np.int32)


def _uniforms(case, seed):
    return np.random.default_rng(seed + 1).random((case["n"], lede.SAMPLE_STRIDE)).astype(np.float32) * np.float32(0.9999)


def _prepare_model(case, seed):
    m, g = _model(case), _generator(seed)
    policy = case.get("mode") == "policy"
    total = case["ctx"] + case["n"] + 16
    eng = lede.Engine(m, max_ctx=total, k_max=15, exit_hidden=POLICY_HIDDEN if policy else 0)
    eng.kv.zero_()
    w, succ = _weights(m, g)
    q, e = _qnets(m, seed)
    eng.lede_load_weights(w, qnet=q, exit_qnet=e if policy else None, n_layers=m.n_layers)
    tokens = _tokens(case, m, g)
    s = {"case": case, "m": m, "eng": eng, "ctx": case["ctx"],
         "logits": torch.empty(16 * m.vocab, dtype=torch.float32, pin_memory=True)}
    eng.lede_set_options(0, 1)  # the logits are read back
    half = eng.region_bytes[1] // 2
    dt = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    es = 2 if m.dtype == "bf16" else 4
    n_pages = eng.cfg.n_pages
    size = m.n_layers * n_pages * m.n_kv_heads * 64 * m.head_dim * es
    last = case["ctx"] + case["n"] - 1
    pages = slice(case["ctx"] // 64, last // 64 + 1)
    for name, at in (("k", 0), ("v", half)):
        s[name] = eng.kv[at:at + size].view(dt).view(m.n_layers, n_pages, m.n_kv_heads, 64, m.head_dim)[:, pages]
    if case["ctx"]:
        eng.lede_prefill(tokens[:case["ctx"]])
    if case["kind"] == "prefill":
        s["new"] = np.ascontiguousarray(tokens[case["ctx"]:])
    else:
        s["first"] = int(succ[int(tokens[-1])])
        s["uniforms"] = _uniforms(case, seed)
    return s


def _prepare_linear(case, seed):
    g = _generator(seed)
    L, N, K, M = lede.load(), case["n_out"], case["n_in"], case["rows"]
    ldx = -(-K // 32) * 32
    w = torch.empty((N, K), dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    x = torch.zeros((M, ldx), dtype=torch.bfloat16, device="cuda")
    x[:, :K] = torch.empty((M, K), dtype=torch.bfloat16, device="cuda").normal_(0.0, 1.0, generator=g)
    tiled = torch.empty(L.lede_op_tiled_bytes(1, N, K), dtype=torch.uint8, device="cuda")
    s = {"case": case, "L": L, "tiled": tiled, "x": x, "ldx": ldx, "y": torch.empty((M, N), dtype=torch.float32, device="cuda")}
    rc = L.lede_op_repack(1, w.data_ptr(), N, K, tiled.data_ptr(), _stream())
    assert rc == 0
    torch.cuda.synchronize()
    s["w"] = w if case.get("keep") else None
    return s


def _sample_inputs(case, seed):
    g = _generator(seed)
    z = torch.empty((case["rows"], case["vocab"]), dtype=torch.float32, device="cuda").normal_(0.0, 2.0, generator=g)
    u = np.random.default_rng(seed).random(case["rows"]).astype(np.float32) * np.float32(0.9999)
    return z, u


def _update_inputs(case, seed):
    r = np.random.default_rng(seed)
    H, B = case["hidden"], case["batch"]
    t = np.zeros((2048, 6), np.float32)
    t[:, :3] = 2.0 * r.standard_normal((2048, 3))
    t[:, 3] = r.integers(0, 2, 2048)
    t[:, 4] = r.standard_normal(2048)
    t[:, 5] = r.random(2048) < 0.15
    init = r.random(6 * H + 2).astype(np.float32)
    u = (r.integers(0, 1 << 24, B) / float(1 << 24)).astype(np.float32)
    noise = r.standard_normal((2, 2 * H + 5)).astype(np.float32)
    return t, init, u, noise


def _prepare_update(case, seed):
    t, init, u, noise = _update_inputs(case, seed)
    q = lede.Dqn(hidden=case["hidden"], capacity=2048, batch=case["batch"], n_step=case["n_step"])
    q.lede_dqn_init(init)
    q.lede_dqn_push(t)
    n = lede.dqn_param_count(case["hidden"])
    step = -(-n * 4 // 256) * 64  # the region's arrays are 256-byte aligned: online, target, Adam m and v
    f = q.region.view(torch.float32)
    s = {"case": case, "q": q, "u": torch.from_numpy(u).cuda(), "noise": torch.from_numpy(noise).cuda()}
    for i, name in enumerate(("online", "target", "m", "v")):
        s[name] = f[i * step:i * step + n]
    return s


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("prefill", "decode"):
        return _prepare_model(case, seed)
    if kind == "linear":
        return _prepare_linear(case, seed)
    if kind == "sample":
        z, u = _sample_inputs(case, seed)
        return {"case": case, "z": z, "u": u}
    return _prepare_update(case, seed)


# ---- one pass --------------------------------------------------------------------------------


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _read_logits(s):
    """The logits rows of the last verify or prefill head, into the pinned buffer."""
    eng, rows, buf = s["eng"], ctypes.c_int32(), s["logits"]
    rc = eng.L.lede_debug_logits(eng.ctx, lede.LOGITS_VERIFY, ctypes.cast(buf.data_ptr(), ctypes.POINTER(ctypes.c_float)),
                                 buf.numel(), ctypes.byref(rows), eng.stream)
    if rc:
        raise RuntimeError("lede_debug_logits: %d" % rc)
    return buf[:rows.value * s["m"].vocab].view(rows.value, s["m"].vocab)


def _run_decode(s):
    case, eng = s["case"], s["eng"]
    n, mode, act = case["n"], case["mode"], (case["l"], case["k"])
    eng.lede_truncate(s["ctx"])
    eng.lede_set_pending(s["first"])
    out, i, q = [], 0, 0.0
    while len(out) < n:
        left = n - len(out)
        if mode == "policy":
            rec = eng.lede_step_policy(left)
        elif mode == "sampled":
            rec = eng.lede_step_sampled(act, TEMPERATURE, s["uniforms"][i], left, False)
        else:
            rec = eng.lede_step(act, left, mode == "ssd")
        if rec.q_action >= 0:
            q = rec.q_max
        out.extend(rec.emitted)
        i += 1
    return {"tokens": np.array(out, np.int32), "q": float(q), "logits": _read_logits(s), "k": s["k"], "v": s["v"]}


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "prefill":
        s["eng"].lede_truncate(s["ctx"])
        token = s["eng"].lede_prefill(s["new"])
        return {"token": token, "logits": _read_logits(s)[-1:], "k": s["k"], "v": s["v"]}
    if kind == "decode":
        return _run_decode(s)
    if kind == "linear":
        rc = s["L"].lede_op_linear(1, s["tiled"].data_ptr(), case["n_out"], case["n_in"], s["x"].data_ptr(), s["ldx"], case["rows"],
                                   s["y"].data_ptr(), 1, _stream())
        if rc:
            raise RuntimeError("lede_op_linear: %d" % rc)
        return s["y"]
    if kind == "sample":
        return np.array(lede.op_sample_noalloc(s["z"], TEMPERATURE, s["u"]), np.int32)
    s["q"].lede_dqn_update(s["u"], s["noise"], want_loss=False)
    return {name: s[name] for name in ("online", "target", "m", "v")}


# ---- what a pass cannot do without -------------------------------------------------------------


def _steps(case):
    """(drafts, rows of the verify) of each step when every draft is accepted."""
    left, steps = case["n"], []
    while left > 0:
        k = min(case["k"], left - 1)
        steps.append(k)
        left -= k + 1
    return steps


def work(case):
    kind = case["kind"]
    if kind == "update":
        P, H, B, n = 6 * case["hidden"] + 2, case["hidden"], case["batch"], case["n_step"]
        return {"bytes": 4 * (2 * P * 7 + B + 2 * (2 * H + 5)) + B * (n + 1) * 24, "flops": B * 20 * P + 30 * 2 * P}
    if kind == "sample":
        return {"bytes": case["rows"] * (case["vocab"] * 4 + 8), "flops": case["rows"] * case["vocab"] * 4}
    if kind == "linear":
        N, K, M = case["n_out"], case["n_in"], case["rows"]
        return {"bytes": 2 * N * K + 2 * M * K + 4 * M * N, "flops": 2 * N * K * M}
    m = _model(case)
    es = 2 if m.dtype == "bf16" else 4
    layer, head, L = _layer_params(m), m.vocab * m.d_model, m.n_layers
    kv = 2 * m.n_kv_heads * m.head_dim * es
    pair = 4 * m.n_heads * m.head_dim  # flops of one query against one key and value
    if kind == "prefill":
        c, n = case["ctx"], case["n"]
        return {"bytes": es * (L * layer + head) + L * (c + n) * kv + n * m.d_model * es + 4 * m.vocab,
                "flops": 2 * n * L * layer + 2 * head + L * pair * (n * c + n * (n + 1) // 2)}
    nbytes = flops = 0
    c, l = case["ctx"], case["l"]
    for k in _steps(case):
        nbytes += k * (es * (l * layer + head) + l * c * kv) + es * (L * layer + head) + L * (c + k + 1) * kv
        flops += k * (2 * (l * layer + head) + l * c * pair) + (k + 1) * (2 * (L * layer + head) + L * c * pair)
        c += k + 1
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Measured against 64-bit results, whose intermediate values aren't rounded: bf16 models are within 1e-2 of them, fp32 ones
    within 1e-5.  Sums in another order move bf16 outputs by about half of that, through the roundings between layers."""
    kind = case["kind"]
    if kind == "update":
        return {"rel": 1e-5, "max": 1e-3}
    if kind == "sample":
        return {"rel": 0.0, "differ": 0.01}
    if kind == "linear":
        return {"rel": 5e-6, "max": 5e-5}
    if case["shape"] == "tiny":
        return {"rel": 2e-5, "max": 2e-4, "differ": 0.01}
    return {"rel": 2e-2, "max": 0.5, "differ": 0.01}


# ---- 64-bit results ------------------------------------------------------------------------------


def _norm(x, gain):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + EPS) * gain.double()


def _layer(x, w, m, cos, sin, first):
    """One decoder layer over all positions of x (rows before `first` are only keys and values of later ones when first > 0 and the
    layer is the last, which the caller doesn't use)."""
    T, hd, G = x.shape[0], m.head_dim, m.n_heads // m.n_kv_heads
    a = _norm(x, w["attn_norm"])

    def rot(y):
        y = y.view(T, -1, hd)
        y0, y1 = y[..., :hd // 2], y[..., hd // 2:]
        return torch.cat([y0 * cos - y1 * sin, y1 * cos + y0 * sin], -1)

    q, k = rot(a @ w["wq"].double().T), rot(a @ w["wk"].double().T)
    v = (a @ w["wv"].double().T).view(T, -1, hd)
    del a
    o = torch.empty_like(q)
    mask = torch.ones((T, T), dtype=torch.bool, device=x.device).triu_(1)
    for h in range(m.n_heads):
        z = (q[:, h] @ k[:, h // G].T) / math.sqrt(hd)
        z.masked_fill_(mask, -math.inf)
        o[:, h] = torch.softmax(z, -1) @ v[:, h // G]
    x = x + o.view(T, -1) @ w["wo"].double().T
    a = _norm(x, w["ffn_norm"])
    x = x + (torch.nn.functional.silu(a @ w["wg"].double().T) * (a @ w["wu"].double().T)) @ w["wd"].double().T
    return x, k, v


def _exact_model(case, seed):
    m, g = _model(case), _generator(seed)
    if case["ctx"] + case["n"] > 4300:
        return None
    w, succ = _weights(m, g)
    tokens = _tokens(case, m, g)
    decode = case["kind"] == "decode"
    chain = []
    if decode:
        t = int(succ[int(tokens[-1])])
        first = t
        for _ in range(case["n"]):
            t = int(succ[t])
            chain.append(t)
        tokens = np.concatenate([tokens, np.array([first] + chain[:-1], np.int32)])
    T = len(tokens)
    x = w["embed"][torch.from_numpy(tokens).long().cuda()].double()
    ang = torch.arange(T, device="cuda").double()[:, None] * m.rope_base ** (-2.0 * torch.arange(m.head_dim // 2, device="cuda").double() / m.head_dim)
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    rows = _steps(case)[-1] + 1 if decode else 1
    steps = _steps(case) if decode else []
    pages = slice(case["ctx"] // 64, (T - 1) // 64 + 1)
    n_pages = (T - 1) // 64 + 1
    out = {n: torch.zeros((m.n_layers, n_pages, m.n_kv_heads, 64, m.head_dim), dtype=torch.float64, device="cuda") for n in "kv"}
    state = None
    for j, lw in enumerate(w["layers"]):
        x, k, v = _layer(x, lw, m, cos, sin, 0)
        for name, y in (("k", k), ("v", v)):
            y = torch.nn.functional.pad(y, (0, 0, 0, 0, 0, n_pages * 64 - T))
            out[name][j] = y.view(n_pages, 64, m.n_kv_heads, m.head_dim).transpose(1, 2)
        if j + 1 == m.exits[0]:
            state = x
        lw.clear()
    logits = _norm(x[T - rows:], w["final_norm"]) @ w["head"].double().T
    res = {"logits": logits, "k": out["k"][:, pages], "v": out["v"][:, pages]}
    if not decode:
        return dict(res, token=int(succ[int(tokens[-1])]))
    qv = 0.0
    if case["mode"] == "ssd":
        # the Q-network sees the pending token of the last step that drafts
        at, pos = case["ctx"], None
        for kk in steps:
            if kk > 0:
                pos = at
            at += kk + 1
        if pos is not None and m.exits[0] <= case["l"]:
            q = {n: torch.from_numpy(a).double().cuda() for n, a in _qnets(m, seed)[0].items()}
            s = _norm(state[pos], w["final_norm"])
            qv = float((q["w2"] @ torch.relu(q["w1"] @ s + q["b1"]) + q["b2"]).max())
    return dict(res, tokens=np.array(chain, np.int32), q=qv)


def _exact_update(case, seed):
    t, init, u, noise = _update_inputs(case, seed)
    H, B, n, gamma, lr, sigma0 = case["hidden"], case["batch"], case["n_step"], 0.99, 6.25e-5, 0.1
    P = 6 * H + 2
    init = torch.from_numpy(init).double()
    fan = torch.full((P,), float(H), dtype=torch.float64)
    fan[:4 * H] = 3.0
    theta = torch.cat([(2 * init - 1) / fan.sqrt(), sigma0 / fan.sqrt()])
    target = theta.clone()
    theta.requires_grad_(True)
    f = lambda e: torch.sign(e) * e.abs().sqrt()  # noqa: E731

    def net(th, eps, s):
        e = f(torch.from_numpy(eps).double())
        i1, o1, i2, o2 = e[:3], e[3:3 + H], e[3 + H:3 + 2 * H], e[3 + 2 * H:]
        scale = torch.cat([torch.outer(o1, i1).flatten(), o1, torch.outer(o2, i2).flatten(), o2])
        w = th[:P] + th[P:] * scale
        hid = torch.relu(s @ w[:3 * H].view(H, 3).T + w[3 * H:4 * H])
        return hid @ w[4 * H:6 * H].view(2, H).T + w[6 * H:]

    tt = torch.from_numpy(t).double()
    pos = (u.astype(np.float64) * (len(t) - n)).astype(np.int64)
    y = torch.zeros(B, dtype=torch.float64)
    boot = net(target, noise[1], tt[pos + n, :3]).max(1).values
    for b, p in enumerate(pos):
        ended = False
        for k in range(n):
            y[b] += gamma ** k * tt[p + k, 4]
            if t[p + k, 5]:
                ended = True
                break
        if not ended:
            y[b] += gamma ** n * boot[b]
    q = net(theta, noise[0], tt[pos, :3])[torch.arange(B), tt[pos, 3].long()]
    ((q - y.detach()) ** 2).mean().backward()
    gr = theta.grad
    m, v = 0.1 * gr, 0.001 * gr * gr
    online = theta.detach() - lr * (m / 0.1) / ((v / 0.001).sqrt() + 1.5e-4)
    return {"online": online, "target": target, "m": m, "v": v}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("prefill", "decode"):
        return _exact_model(case, seed)
    if kind == "update":
        return _exact_update(case, seed)
    if kind == "sample":
        z, u = _sample_inputs(case, seed)
        w = torch.softmax(z.double() / float(np.float32(TEMPERATURE)), -1).cumsum(-1)
        at = torch.searchsorted(w, (torch.from_numpy(u).double().cuda() * w[:, -1])[:, None], right=True)
        return at[:, 0].int()
    s = _prepare_linear(dict(case, keep=True), seed)
    return s["x"][:, :case["n_in"]].double() @ s["w"].double().T
