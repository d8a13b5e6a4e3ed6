"""Performance cases of the Speculative Rejection library on one MI355X.

Each case is one pass through public entry points of paper_2410_20290_amd, on
inputs made on the GPU from a seed.  The shapes are the repository's own
configurations (tiny fp32, small, 1B and 8B bf16; the 1B and 8B shapes with
few layers, since their layers repeat) and the row counts, prompt lengths and
response lengths that their runs go through:

  generate        a whole sr_generate call (prefill, decode, sampling, scoring,
                  cuts, answer)
  decode          the generator's decode loop over given tokens: logits of
                  every response position
  reward          the reward model's scoring pass over partial responses
  layer           the four projections of one decoder layer
  decode_attn     decode attention over a shared prefix and per-row tails
  prefill_attn    causal attention of new tokens after cached ones
  sample          the next-token draw over the vocabulary
  cut             the selection of the survivors and their KV compaction
"""
import math

import numpy as np
import torch

import paper_2410_20290_amd as sr
import synth

BASE = {
    "tiny": synth.CONFIGS["tiny_fp32"].model,
    "small": synth.CONFIGS["small_bf16"].model,
    "1b": synth.CONFIGS["1b_bf16"].model,
    "8b": synth.CONFIGS["8b_bf16"].model,
}


def listed():
    return [
        # one short prompt on the tiny fp32 pair: host work, launches and
        # round trips are all there is
        {"name": "generate_tiny", "kind": "generate", "shape": "tiny", "P": 32, "n": 16, "tau": 16, "alpha": 0.5,
         "max_new": 64},
        # decode steps of a small model: a chain of short launches
        {"name": "decode_small_64", "kind": "decode", "shape": "small", "layers": 4, "P": 128, "rows": 64, "len": 32},
        # decode steps after the first cut of an 8B run (N = 512, alpha 0.8)
        {"name": "decode_8b_103", "kind": "decode", "shape": "8b", "layers": 2, "P": 256, "rows": 103, "len": 9},
        # the first decision of an 8B run: 512 partial responses of 128 tokens
        {"name": "reward_8b_512x128", "kind": "reward", "shape": "8b", "layers": 2, "P": 256, "rows": 512, "len": 128},
        # the projections of a late decode step: few survivors, weight-bound
        {"name": "layer_8b_21", "kind": "layer", "shape": "8b", "rows": 21},
        # the projections of a first-round decode step: the whole batch
        {"name": "layer_8b_512", "kind": "layer", "shape": "8b", "rows": 512},
        # a prompt of odd length through one layer of the 1B shape
        {"name": "layer_1b_771", "kind": "layer", "shape": "1b", "rows": 771},
        # decode attention in the first round of an 8B run, near its end
        {"name": "decode_attn_8b_512", "kind": "decode_attn", "shape": "8b", "rows": 512, "P": 256, "lt": 101},
        # decode attention of a few long survivors, head_dim 64
        {"name": "decode_attn_1b_37", "kind": "decode_attn", "shape": "1b", "rows": 37, "P": 256, "lt": 699},
        # the second scoring round of an 8B run: new tokens after cached ones
        {"name": "prefill_attn_8b_103", "kind": "prefill_attn", "shape": "8b", "rows": 103, "P": 256, "t0": 128,
         "lr": 507},
        # one draw for the whole batch over the 8B vocabulary
        {"name": "sample_512x128256", "kind": "sample", "rows": 512, "vocab": 128256, "temperature": 1.0},
        # a first cut: a fifth of 512 rows survive; four layers' keys and
        # values of 128 tokens are packed
        {"name": "cut_8b_512", "kind": "cut", "shape": "8b", "layers": 4, "rows": 512, "keep": 103, "len": 127,
         "cap_dst": 636},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["generate", "decode", "decode", "reward", "reward", "layer", "layer", "layer", "decode_attn",
                       "decode_attn", "prefill_attn", "prefill_attn", "sample", "cut"])
    if kind == "generate":
        tau = rng.randint(6, 20)
        return {"kind": kind, "shape": "tiny", "P": _log(rng, 5, 70), "n": rng.randint(4, 24), "tau": tau,
                "alpha": rng.choice([0.0, 0.5, 0.6, 0.75, 0.8, 0.9]), "max_new": rng.randint(2 * tau, 64)}
    if kind == "decode":
        shape = rng.choice(["tiny", "small", "1b", "8b"])
        rows = _log(rng, 3, 512)
        return {"kind": kind, "shape": shape, "layers": {"tiny": 2, "small": 4}.get(shape, 2), "P": _log(rng, 20, 512),
                "rows": rows, "len": max(3, min(24, 1200 // rows))}
    if kind == "reward":
        shape = rng.choice(["small", "1b", "8b"])
        rows = _log(rng, 4, 256)
        return {"kind": kind, "shape": shape, "layers": {"small": 4}.get(shape, 2), "P": _log(rng, 20, 512), "rows": rows,
                "len": min(512, _log(rng, 16, max(17, 30000 // rows)))}
    if kind == "layer":
        shape = rng.choice(["tiny", "small", "1b", "8b", "8b"])
        return {"kind": kind, "shape": shape, "rows": _log(rng, 1, {"8b": 9000, "1b": 20000}.get(shape, 3000))}
    if kind == "decode_attn":
        shape = rng.choice(["tiny", "small", "1b", "8b", "8b"])
        rows = _log(rng, 3, 1024)
        return {"kind": kind, "shape": shape, "rows": rows, "P": _log(rng, 16, 512),
                "lt": min(1024, _log(rng, 2, max(8, 200000 // rows)))}
    if kind == "prefill_attn":
        shape = rng.choice(["tiny", "small", "1b", "8b", "8b"])
        rows = 1 if rng.random() < 0.25 else _log(rng, 2, 256)
        lr = min(640, _log(rng, 24, max(32, 50000 // rows)))
        return {"kind": kind, "shape": shape, "rows": rows, "P": 0 if rows == 1 else _log(rng, 16, 512),
                "t0": 0 if rows == 1 else rng.choice([0, rng.randint(1, 300)]), "lr": lr}
    if kind == "sample":
        return {"kind": kind, "rows": _log(rng, 1, 1024), "vocab": rng.choice([512, 8192, 32000, 50257, 128256]),
                "temperature": rng.choice([0.0, 0.7, 1.0, 1.0])}
    shape = rng.choice(["tiny", "small", "1b", "8b"])
    rows = _log(rng, 8, 600)
    ln = rng.randint(7, 250)
    return {"kind": kind, "shape": shape, "layers": 2, "rows": rows, "keep": max(1, int(rows * rng.uniform(0.1, 0.6))),
            "len": ln, "cap_dst": ln + rng.randint(1, 300)}


# ---------------------------------------------------------------- inputs
def _shape(case):
    b = BASE[case["shape"]]
    return synth.ModelShape(case.get("layers", b.n_layers), b.d_model, b.n_heads, b.n_kv_heads, b.head_dim, b.ffn_dim,
                            b.vocab, b.dtype, b.rope_theta, b.rms_eps)


def _dtype(m):
    return torch.bfloat16 if m.dtype == "bf16" else torch.float32


def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * int(seed) + 17)
    return g


def _randn(g, shape, std, dtype, mean=0.0):
    t = torch.empty(shape, dtype=dtype, device="cuda")
    return t.normal_(mean, std, generator=g)


def _model(g, m, reward):
    """Random weights on the device and their descriptor."""
    ts = {}
    for name, shape in synth.weight_shapes(m, reward).items():
        ts[name] = _randn(g, shape, 0.1, _dtype(m), 1.0) if name.endswith("norm") else _randn(g, shape, 0.02, _dtype(m))
    cfg = sr.sr_model_config(m.n_layers, m.d_model, m.n_heads, m.n_kv_heads, m.head_dim, m.ffn_dim, m.vocab,
                             m.rope_theta, m.rms_eps, sr.SR_BF16 if m.dtype == "bf16" else sr.SR_F32, int(reward))
    w = sr.sr_weights(*[ts[n].data_ptr() for n in ("embed", "attn_norm", "wqkv", "wo", "ffn_norm", "w13", "w2",
                                                   "final_norm", "head")])
    return sr.DeviceModel(m, reward, ts, sr.sr_model(cfg, w))


def _tokens(g, shape, vocab):
    return torch.randint(0, vocab, shape, generator=g, device="cuda", dtype=torch.int32)


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    if kind in ("generate", "decode", "reward"):
        m = _shape(case)
        gen, rm = _model(g, m, False), _model(g, m, True)
        prompt = _tokens(g, (case["P"],), m.vocab).cpu().numpy()
        st = {"case": case, "gen": gen, "rm": rm, "prompt": prompt}
        if kind == "generate":
            st["p"] = sr.make_params(case["n"], case["alpha"], case["tau"], case["max_new"], 1.0, 42 + int(seed))
        else:
            st["p"] = sr.make_params(case["rows"], 0.8, case["len"], case["len"])
            st["tokens"] = _tokens(g, (case["rows"], case["len"]), m.vocab)
            lens = torch.randint(max(1, case["len"] - 7), case["len"] + 1, (case["rows"],), generator=g, device="cuda",
                                 dtype=torch.int32)
            st["lens"] = lens
        st["ws"] = sr.Workspace(gen, rm, case["P"], st["p"])
        return st
    if kind == "layer":
        m = _shape(case)
        dt, M = _dtype(m), case["rows"]
        qd = m.n_heads * m.head_dim
        return {"case": case,
                "x": _randn(g, (M, m.d_model), 1.0, dt), "a": _randn(g, (M, qd), 0.5, dt),
                "f": _randn(g, (M, m.d_model), 1.0, dt), "h": _randn(g, (M, m.d_model), 1.0, torch.float32),
                "wqkv": _randn(g, (m.qkv_dim, m.d_model), 0.02, dt), "wo": _randn(g, (m.d_model, qd), 0.02, dt),
                "w13": _randn(g, (2, m.ffn_dim, m.d_model), 0.02, dt), "w2": _randn(g, (m.d_model, m.ffn_dim), 0.02, dt),
                "qkv": torch.empty((M, m.qkv_dim), dtype=torch.float32, device="cuda"),
                "o": torch.empty((M, m.d_model), dtype=torch.float32, device="cuda"),
                "u": torch.empty((M, m.ffn_dim), dtype=dt, device="cuda")}
    if kind == "decode_attn":
        m = _shape(case)
        dt, R, hk, hd = _dtype(m), case["rows"], m.n_kv_heads, m.head_dim
        cap = case["lt"] + 3
        return {"case": case, "q": _randn(g, (R, m.n_heads, hd), 1.2, torch.float32),
                "kp": _randn(g, (hk, case["P"], hd), 1.2, dt), "vp": _randn(g, (hk, case["P"], hd), 1.0, dt),
                "kt": _randn(g, (R, hk, cap, hd), 1.2, dt), "vt": _randn(g, (R, hk, cap, hd), 1.0, dt),
                "out": torch.empty((R, m.n_heads * hd), dtype=dt, device="cuda")}
    if kind == "prefill_attn":
        m = _shape(case)
        dt, R, hk, hd, P = _dtype(m), case["rows"], m.n_kv_heads, m.head_dim, case["P"]
        cap = case["t0"] + case["lr"]
        return {"case": case, "q": _randn(g, (R, case["lr"], m.n_heads, hd), 1.2, torch.float32),
                "kp": _randn(g, (hk, P, hd), 1.2, dt) if P else None, "vp": _randn(g, (hk, P, hd), 1.0, dt) if P else None,
                "ko": _randn(g, (R, hk, cap, hd), 1.2, dt), "vo": _randn(g, (R, hk, cap, hd), 1.0, dt),
                "out": torch.empty((R, case["lr"], m.n_heads * hd), dtype=dt, device="cuda")}
    if kind == "sample":
        R = case["rows"]
        return {"case": case, "seed": 42 + int(seed), "logits": _randn(g, (R, case["vocab"]), 1.3, torch.float32),
                "cand": torch.randperm(4096, generator=g, device="cuda")[:R].to(torch.int32),
                "tok": torch.empty(R, dtype=torch.int32, device="cuda")}
    m = _shape(case)
    R, ln, es = case["rows"], case["len"], 2 if m.dtype == "bf16" else 4
    row = m.n_kv_heads * m.head_dim
    sb, db = R * row * ln, R * row * case["cap_dst"]
    it = torch.int16 if es == 2 else torch.int32
    return {"case": case, "m": m, "es": es, "sb": sb, "db": db,
            "scores": _randn(g, (R,), 1.0, torch.float32),
            "cand": torch.randperm(4096, generator=g, device="cuda")[:R].to(torch.int32).sort().values,
            "src": torch.randint(-30000, 30000, (2 * m.n_layers * sb,), generator=g, device="cuda", dtype=it),
            "dst": torch.zeros(2 * m.n_layers * db, dtype=it, device="cuda"),
            "accept": torch.empty(R, dtype=torch.int32, device="cuda"),
            "src_row": torch.zeros(R, dtype=torch.int32, device="cuda"),
            "count": torch.zeros(1, dtype=torch.int32, device="cuda")}


def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "generate":
        out = sr.generate(st["gen"], st["rm"], st["prompt"], st["p"], st["ws"], trace=True, max_rounds_cap=8)
        return {"tokens": np.asarray(out["tokens"], dtype=np.int32), "score": np.float32([out["best_score"]]),
                "final_scores": out["trace"]["final_scores"], "round_scores": out["trace"]["round_scores"]}
    if kind == "decode":
        return sr.logits_teacher_forced(st["gen"], st["rm"], st["prompt"], st["p"], st["tokens"], st["ws"])
    if kind == "reward":
        return sr.reward_scores(st["gen"], st["rm"], st["prompt"], st["p"], st["tokens"], st["lens"], st["ws"])
    if kind == "layer":
        h = st["h"].clone()  # the residual stream before the layer stays what it was
        sr.projection(st["x"], st["wqkv"], 0, st["qkv"])
        sr.projection(st["a"], st["wo"], 0, st["o"])
        sr.projection(st["f"], st["w13"], 2, st["u"])
        sr.projection(st["u"], st["w2"], 1, h)
        return {"qkv": st["qkv"], "o": st["o"], "u": st["u"], "h": h}
    if kind == "decode_attn":
        sr.decode_attention(st["q"], st["kp"], st["vp"], st["kt"], st["vt"], case["lt"], st["out"])
        return st["out"]
    if kind == "prefill_attn":
        sr.prefill_attention(st["q"], st["kp"], st["vp"], st["ko"], st["vo"], case["t0"], st["out"])
        return st["out"]
    if kind == "sample":
        sr.sample(st["logits"], st["cand"], 7, case["temperature"], st["seed"], st["tok"])
        return st["tok"]
    m = st["m"]
    sr.select(st["scores"], st["cand"], case["keep"], st["accept"])
    sr.compact(st["src"], st["sb"], st["dst"], st["db"], st["accept"], m.n_layers, m.n_kv_heads, m.head_dim, st["es"],
               case["len"], case["cap_dst"], case["len"], st["src_row"], st["count"])
    return {"accept": st["accept"], "count": st["count"], "dst": st["dst"]}


# ------------------------------------------------------------ what a pass needs
def _keep(b, alpha):
    return b - (int(math.floor(alpha * 1e6 + 0.5)) * b) // 1000000


def _schedule(case):
    """[(rows, first step, decision length)] of a generate call without EOS."""
    b, L, out = case["n"], 0, []
    budget = case["n"] * case["tau"]
    while True:
        D = case["max_new"] if _keep(b, case["alpha"]) == b else min(case["max_new"], budget // b)
        if D > L:
            out.append((b, L, D))
            L = D
        if L == case["max_new"]:
            return out
        b = _keep(b, case["alpha"])


def _layer_elems(m):
    return m.qkv_dim * m.d_model + m.d_model * m.n_heads * m.head_dim + 3 * m.ffn_dim * m.d_model


def _tokens_work(m, T, keys):
    """flops of T tokens through the layers, each attending `keys` on average."""
    return 2.0 * T * m.n_layers * _layer_elems(m) + 4.0 * T * m.n_layers * m.n_heads * m.head_dim * keys


def work(case):
    kind = case["kind"]
    if kind in ("generate", "decode", "reward"):
        m = _shape(case)
        es = 2 if m.dtype == "bf16" else 4
        wl, P = float(m.n_layers * _layer_elems(m) * es), case["P"]
        kv = 2.0 * m.n_layers * m.n_kv_heads * m.head_dim * es  # bytes of one token's keys and values
        head = m.vocab * m.d_model
        by, fl = wl, _tokens_work(m, P, P / 2)

        def steps(rows, a, b):
            n = b - a
            mean = (a + b) / 2
            return (n * (wl + head * es + kv * (P + rows * mean) + 4.0 * rows * m.vocab),
                    _tokens_work(m, rows * n, P + mean) + 2.0 * rows * n * head)

        if kind == "decode":
            s = steps(case["rows"], 1, case["len"])
            return {"bytes": by + s[0], "flops": fl + s[1]}
        if kind == "reward":
            T, ln = case["rows"] * case["len"], case["len"]
            act = 4.0 * T * m.d_model
            return {"bytes": 2 * by + kv * (P + T) + act, "flops": fl + _tokens_work(m, T, P + ln / 2)}
        by, fl = 2 * by, 2 * fl
        for b, a, D in _schedule(case):
            s = steps(b, max(a, 1), D)
            by += s[0] + wl + kv * b * (D - a)
            fl += s[1] + _tokens_work(m, b * (D - a), P + D / 2)
        return {"bytes": by, "flops": fl}
    if kind == "layer":
        m = _shape(case)
        M, es = case["rows"], 2 if m.dtype == "bf16" else 4
        qd = m.n_heads * m.head_dim
        ins = M * (2 * m.d_model + qd) * es + 4.0 * M * m.d_model
        outs = 4.0 * M * (m.qkv_dim + 2 * m.d_model) + es * M * m.ffn_dim
        return {"bytes": ins + outs + es * _layer_elems(m), "flops": 2.0 * M * _layer_elems(m)}
    if kind == "decode_attn":
        m = _shape(case)
        es, R, hq, hd = 2 if m.dtype == "bf16" else 4, case["rows"], m.n_heads, m.head_dim
        keys = case["P"] + R * case["lt"]
        return {"bytes": 2.0 * m.n_kv_heads * hd * es * keys + R * hq * hd * (4.0 + es),
                "flops": 4.0 * R * hq * hd * (case["P"] + case["lt"])}
    if kind == "prefill_attn":
        m = _shape(case)
        es, R, hq, hd, lr = 2 if m.dtype == "bf16" else 4, case["rows"], m.n_heads, m.head_dim, case["lr"]
        keys = case["P"] + R * (case["t0"] + lr)
        return {"bytes": 2.0 * m.n_kv_heads * hd * es * keys + R * lr * hq * hd * (4.0 + es),
                "flops": 4.0 * R * hq * hd * ((case["P"] + case["t0"]) * lr + lr * (lr + 1) / 2)}
    if kind == "sample":
        return {"bytes": 4.0 * case["rows"] * case["vocab"], "flops": 4.0 * case["rows"] * case["vocab"]}
    m = _shape(case)
    es = 2 if m.dtype == "bf16" else 4
    moved = 4.0 * m.n_layers * case["keep"] * case["len"] * m.n_kv_heads * m.head_dim * es
    return {"bytes": moved + 12.0 * case["rows"], "flops": 0.0}


def tolerance(case):
    """About four times the error measured against the 64-bit results: 2e-6
    for the fp32 model's scores, 2e-3 for a layer's bf16 outputs, 3e-3 for
    bf16 attention, 5e-3 for four small bf16 layers, 1.1e-2 for two layers of
    the 8B shape."""
    kind = case["kind"]
    if kind in ("sample", "cut"):
        return "exact"
    if case["shape"] == "tiny":
        return {"rel": 1e-5}
    if kind == "layer":
        return {"rel": 7e-3}
    if kind in ("decode_attn", "prefill_attn"):
        return {"rel": 1.2e-2}
    return {"rel": 2e-2 if case["shape"] == "small" else 3e-2}


# ------------------------------------------------------------ 64-bit results
def _norm64(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g.double()


def _rope64(x, pos0, theta):
    """x [R][T][heads][hd], positions pos0 + t; rotates halves."""
    hd, T = x.shape[-1], x.shape[1]
    half = hd // 2
    f = theta ** (-2.0 * torch.arange(half, dtype=torch.float64, device=x.device) / hd)
    a = (pos0 + torch.arange(T, dtype=torch.float64, device=x.device))[:, None] * f
    c, s = a.cos()[None, :, None], a.sin()[None, :, None]
    x1, x2 = x[..., :half], x[..., half:]
    return torch.cat([x1 * c - x2 * s, x2 * c + x1 * s], dim=-1)


def _attn64(q, kp, vp, ko, vo, t0):
    """q [R][T][hq][hd] at positions t0 + t after a prefix [hkv][P][hd];
    own keys [R][hkv][t0 + T][hd]."""
    R, T, hq, hd = q.shape
    hkv, own = ko.shape[1], ko.shape[2]
    P = 0 if kp is None else kp.shape[1]
    grp, out = hq // hkv, torch.empty_like(q)
    keep = torch.arange(own, device=q.device)[None, :] <= t0 + torch.arange(T, device=q.device)[:, None]
    keep = torch.cat([torch.ones((T, P), dtype=torch.bool, device=q.device), keep], dim=1)
    per = max(1, int(2.5e8 / (hq * T * (P + own))))
    for r in range(0, R, per):
        n = min(per, R - r)
        k, v = ko[r:r + n].double(), vo[r:r + n].double()
        if P:
            k = torch.cat([kp.double()[None].expand(n, -1, -1, -1), k], dim=2)
            v = torch.cat([vp.double()[None].expand(n, -1, -1, -1), v], dim=2)
        qq = q[r:r + n].reshape(n, T, hkv, grp, hd).permute(0, 2, 3, 1, 4).reshape(n * hkv, grp * T, hd).contiguous()
        kt = k.reshape(n * hkv, P + own, hd).transpose(1, 2).contiguous()
        s = torch.matmul(qq, kt) / math.sqrt(hd)
        s = s.view(n * hkv, grp, T, P + own).masked_fill_(~keep, -math.inf).softmax(-1)
        o = torch.matmul(s.view(n * hkv, grp * T, P + own), v.reshape(n * hkv, P + own, hd).contiguous())
        out[r:r + n] = o.view(n, hkv, grp, T, hd).permute(0, 3, 1, 2, 4).reshape(n, T, hq, hd)
    return out


def _forward64(model, tokens, pos0, prefix=None, chunk=8192):
    """Hidden states [R][T][d] in float64 and the layers' keys and values;
    prefix: the keys and values [hkv][P][hd] of a shared prompt, by layer."""
    m, w = model.shape, model.tensors
    R, T = tokens.shape
    h = w["embed"][tokens.long()].double()
    kv = []
    per = max(1, chunk // T)
    hd, hq, hkv = m.head_dim, m.n_heads, m.n_kv_heads
    for l in range(m.n_layers):
        wq, wo = w["wqkv"][l].double().t(), w["wo"][l].double().t()
        w1, w3, w2 = w["w13"][l, 0].double().t(), w["w13"][l, 1].double().t(), w["w2"][l].double().t()
        for r in range(0, R, per):
            x = h[r:r + per]
            n = x.shape[0]
            qkv = (_norm64(x, w["attn_norm"][l], m.rms_eps) @ wq).view(n, T, hq + 2 * hkv, hd)
            q, k = _rope64(qkv[:, :, :hq], pos0, m.rope_theta), _rope64(qkv[:, :, hq:hq + hkv], pos0, m.rope_theta)
            k, v = k.transpose(1, 2).contiguous(), qkv[:, :, hq + hkv:].transpose(1, 2).contiguous()
            kp, vp = (None, None) if prefix is None else prefix[l]
            x = x + _attn64(q, kp, vp, k, v, 0).reshape(n, T, hq * hd) @ wo
            f = _norm64(x, w["ffn_norm"][l], m.rms_eps)
            h[r:r + per] = x + (torch.nn.functional.silu(f @ w1) * (f @ w3)) @ w2
            if prefix is None:
                kv.append((k[0], v[0]))
    return h, kv


def _prompt64(model, prompt):
    t = torch.from_numpy(prompt).cuda()[None]
    return _forward64(model, t, 0)


def _logits64(model, h):
    return _norm64(h, model.tensors["final_norm"], model.shape.rms_eps) @ model.tensors["head"].double().t()


def _scores64(rm, h, lens):
    x = h[torch.arange(h.shape[0], device=h.device), lens.long() - 1]
    return _norm64(x, rm.tensors["final_norm"], rm.shape.rms_eps) @ rm.tensors["head"].double()


def _philox_word0(t, k, seed):
    """Word 0 of Philox4x32-10 (Salmon et al., SC'11) of counter (t, k, 0, 0)."""
    c, key, mask = [t, k, 0, 0], [seed & 0xFFFFFFFF, seed >> 32], 0xFFFFFFFF
    for _ in range(10):
        p0, p1 = 0xD2511F53 * c[0], 0xCD9E8D57 * c[2]
        c = [(p1 >> 32) ^ c[1] ^ key[0], p1 & mask, (p0 >> 32) ^ c[3] ^ key[1], p0 & mask]
        key = [(key[0] + 0x9E3779B9) & mask, (key[1] + 0xBB67AE85) & mask]
    return c[0]


def _generate64(st):
    case, gen, rm, p = st["case"], st["gen"], st["rm"], st["p"]
    P, n = case["P"], case["n"]
    hg, pre_g = _prompt64(gen, st["prompt"])
    _, pre_r = _prompt64(rm, st["prompt"])
    final, rounds, r = np.full(n, np.nan), np.zeros((8, n)), 0
    cand, toks = list(range(n)), torch.zeros((n, 0), dtype=torch.int32, device="cuda")
    b, L = n, 0
    while True:
        D = case["max_new"] if _keep(b, case["alpha"]) == b else min(case["max_new"], n * case["tau"] // b)
        for t in range(L, D):
            if t == 0:
                lg = _logits64(gen, hg[:, -1]).expand(b, -1)
            else:
                lg = _logits64(gen, _forward64(gen, toks, P, pre_g)[0][:, -1])
            cum = lg.softmax(-1).cumsum(-1)
            u = torch.tensor([_philox_word0(t, k, p.seed) / 2.0 ** 32 for k in cand], dtype=torch.float64, device="cuda")
            nxt = torch.searchsorted(cum.contiguous(), u[:, None] * cum[:, -1:], right=True)
            toks = torch.cat([toks, nxt.to(torch.int32)], dim=1)
        if D > L:
            L = D
            lens = torch.full((b,), L, dtype=torch.int32, device="cuda")
            sc = _scores64(rm, _forward64(rm, toks, P, pre_r)[0], lens).cpu().numpy()
        if L == case["max_new"]:
            break
        rounds[r, :b] = sc
        r += 1
        keep = sorted(sorted(range(b), key=lambda i: (-sc[i], cand[i]))[:_keep(b, case["alpha"])])
        cand, toks, sc, b = [cand[i] for i in keep], toks[keep], sc[keep], len(keep)
    for i, k in enumerate(cand):
        final[k] = sc[i]
    best = int(np.argmax(sc))
    return {"tokens": None, "score": sc[best:best + 1], "final_scores": final, "round_scores": rounds}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("sample", "cut"):
        return None
    st = prepare(case, seed)
    if kind == "generate":
        return _generate64(st)
    if kind == "decode":
        hp, pre = _prompt64(st["gen"], st["prompt"])
        h, _ = _forward64(st["gen"], st["tokens"][:, :-1].contiguous(), case["P"], pre)
        out = torch.empty((case["rows"], case["len"], st["gen"].shape.vocab), dtype=torch.float64, device="cuda")
        out[:, 0] = _logits64(st["gen"], hp[0, -1])
        for t in range(1, case["len"]):
            out[:, t] = _logits64(st["gen"], h[:, t - 1])
        return out
    if kind == "reward":
        _, pre = _prompt64(st["rm"], st["prompt"])
        return _scores64(st["rm"], _forward64(st["rm"], st["tokens"], case["P"], pre)[0], st["lens"])
    if kind == "layer":
        x, a, f, h = (st[k].double() for k in ("x", "a", "f", "h"))
        u = torch.nn.functional.silu(f @ st["w13"][0].double().t()) * (f @ st["w13"][1].double().t())
        return {"qkv": x @ st["wqkv"].double().t(), "o": a @ st["wo"].double().t(), "u": u,
                "h": h + u @ st["w2"].double().t()}
    q = st["q"].double()
    if kind == "decode_attn":
        lt = case["lt"]
        kt, vt = st["kt"][:, :, :lt], st["vt"][:, :, :lt]
        return _attn64(q[:, None], st["kp"], st["vp"], kt, vt, lt - 1).reshape(case["rows"], -1)
    return _attn64(q, st["kp"], st["vp"], st["ko"], st["vo"], case["t0"]).reshape(case["rows"], case["lr"], -1)
