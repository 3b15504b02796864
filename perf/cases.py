"""The performance cases of this framework: the calls that a VLA server makes, over the range it makes them in.

A server holds one or more models and, for every batch of requests, runs the VLM stage (`Model.prefill`: camera
frames and instruction text to the prefix state) and then the action stage (`Model.denoise`: an Euler loop of the
action transformer over that state); in steady state it runs the VLM stage of one batch beside the action stage of
the previous one (`vla.step`). The cases are these three calls, and whole requests (prefill, then denoise) for the
fp32 model. Widths, token counts, horizons and step counts are those of the model configurations in
`paper_2609_12075_amd/synth.py`; the stacks are cut to a few layers, so that a case is the chain of a few blocks
whose rounding can be bounded. Batches run from 1 to each configuration's maximum, and text lengths, horizons and
step counts vary around the configured ones.

Weights, pixels, token ids, noise and (for the action stage alone) the prefix state are drawn on the GPU from the
seed: weights N(0, 0.02) with norm gains around 1, pixels U[0, 1), ids uniform, noise N(0, 1), and prefix keys and
values N(0, s) with the s that a normalised hidden state times such weights has.
"""
import math

import torch

from paper_2609_12075_amd import synth, vla

# ------------------------------------------------------------------ shapes


def _vlm_cfg(c):
    """The VLM stage of a configuration: its widths, `vit` ViT layers and `llm` LLM layers; the action expert that
    the constructor asks for is not run and is kept narrow (for a DiT head, whose cross-attention keys and values
    belong to the VLM stage, the width stays)."""
    b = synth.CONFIGS[c["model"]]
    joint = b.head_kind == synth.HEAD_JOINT
    return b.with_(vit_layers=c["vit"], llm_layers=c["llm"], act_layers=c["llm"] if joint else c["act"],
                   act_d=64 if joint else b.act_d, act_mlp=64, n_text=c["text"], max_batch=c["batch"])


def _act_cfg(c):
    """The action stage of a configuration: its widths and `act` layers; the VLM's MLP and ViT, which the call does
    not touch, are left out."""
    b = synth.CONFIGS[c["model"]]
    joint = b.head_kind == synth.HEAD_JOINT
    # (the vision encoder's token merge needs an encoder: without one its tokens come from the plain configuration)
    return b.with_(vit_layers=0, llm_mlp=64, llm_layers=c["act"] if joint else 1, act_layers=c["act"],
                   n_text=c["text"], horizon=c["horizon"], max_batch=c["batch"])


def _whole_cfg(c):
    return synth.CONFIGS[c["model"]].with_(n_text=c["text"], horizon=c["horizon"], max_batch=c["batch"])


def _lockstep(c):
    """The two halves of a lockstep as cases of their own."""
    v = {"kind": "vlm", "model": c["model"], "batch": c["batch"], "text": c["text"], "vit": c["vit"], "llm": c["llm"],
         "act": 2}
    a = {"kind": "action", "model": c["act_model"], "batch": c["act_batch"], "text": c["text"],
         "horizon": c["horizon"], "steps": c["steps"], "act": c["act"]}
    return v, a


def _cfg(c):
    return {"vlm": _vlm_cfg, "action": _act_cfg, "request": _whole_cfg}[c["kind"]](c)


# ------------------------------------------------------------------ cases


def listed():
    return [
        # one robot on the small fp32 model: the whole request, every kernel a few microseconds
        {"name": "request_tiny_f32_b1", "kind": "request", "model": "tiny", "batch": 1, "text": 16, "horizon": 8,
         "steps": 4},
        # the action stage of a single request: 50 action tokens, launches and latency
        {"name": "action_smolvla_b1", "kind": "action", "model": "smolvla", "batch": 1, "text": 48, "horizon": 50,
         "steps": 10, "act": 4},
        {"name": "action_pi0_b1", "kind": "action", "model": "pi0", "batch": 1, "text": 48, "horizon": 50,
         "steps": 10, "act": 4},
        # the DiT head, a batch that is no power of two
        {"name": "action_gr00t_b3", "kind": "action", "model": "gr00t", "batch": 3, "text": 40, "horizon": 16,
         "steps": 4, "act": 4},
        # the action stage of a full batch: 800 and 400 rows
        {"name": "action_smolvla_b16", "kind": "action", "model": "smolvla", "batch": 16, "text": 48, "horizon": 50,
         "steps": 10, "act": 4},
        {"name": "action_pi0_b8", "kind": "action", "model": "pi0", "batch": 8, "text": 48, "horizon": 50,
         "steps": 10, "act": 4},
        # the VLM stage of a single request, the step a robot waits for
        {"name": "vlm_gr00t_b1", "kind": "vlm", "model": "gr00t", "batch": 1, "text": 40, "vit": 2, "llm": 2,
         "act": 2},
        # the VLM stage of small models: without and with the vision encoder (1024 patch tokens an image)
        {"name": "vlm_smolvla_b4", "kind": "vlm", "model": "smolvla", "batch": 4, "text": 48, "vit": 0, "llm": 4,
         "act": 4},
        {"name": "vlm_smolvla_vit_b3", "kind": "vlm", "model": "smolvla_vit", "batch": 3, "text": 37, "vit": 2,
         "llm": 2, "act": 2},
        # the VLM stage at the serving batch, and the largest call a server makes
        {"name": "vlm_pi0_b8", "kind": "vlm", "model": "pi0", "batch": 8, "text": 48, "vit": 2, "llm": 3, "act": 3},
        {"name": "vlm_pi0_b32", "kind": "vlm", "model": "pi0", "batch": 32, "text": 48, "vit": 2, "llm": 3, "act": 3},
        # a lockstep of two co-located models: the VLM stage on a part of the CUs beside the action stage
        {"name": "lockstep_pi0_b4_smolvla_b8", "kind": "lockstep", "model": "pi0", "batch": 4, "text": 48, "vit": 2,
         "llm": 2, "act_model": "smolvla", "act_batch": 8, "horizon": 50, "steps": 10, "act": 4, "cus": 192},
    ]


def draw(rng):
    def log(lo, hi):
        return min(hi, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))

    def action(model):
        b = synth.CONFIGS[model]
        dit = b.head_kind == synth.HEAD_DIT
        return {"kind": "action", "model": model, "batch": log(1, b.max_batch), "text": rng.randint(8, 96),
                "horizon": rng.randint(8, 32) if dit else rng.randint(10, 50),
                "steps": rng.randint(4, 8) if dit else rng.randint(5, 10), "act": rng.randint(2, 4)}

    def vlm(model):
        b = synth.CONFIGS[model]
        return {"kind": "vlm", "model": model, "batch": log(1, b.max_batch), "text": rng.randint(8, 48),
                "vit": rng.randint(1, 2) if b.vit_layers else 0, "llm": rng.randint(2, 3), "act": 2}

    kind = rng.choice(["action"] * 9 + ["vlm"] * 8 + ["request"] * 2 + ["lockstep"])
    if kind == "action":
        return action(rng.choice(["smolvla", "pi0", "gr00t"]))
    if kind == "vlm":
        return vlm(rng.choice(["smolvla", "smolvla_vit", "pi0", "gr00t"]))
    if kind == "request":
        return {"kind": "request", "model": "tiny", "batch": rng.randint(1, 4), "text": rng.randint(8, 64),
                "horizon": rng.randint(8, 50), "steps": rng.randint(4, 10)}
    v = vlm(rng.choice(["smolvla", "pi0"]))
    a = action("smolvla" if v["model"] == "pi0" else "pi0")
    return {"kind": "lockstep", "model": v["model"], "batch": min(8, v["batch"]), "text": v["text"], "vit": v["vit"],
            "llm": v["llm"], "act_model": a["model"], "act_batch": min(8, a["batch"]), "horizon": a["horizon"],
            "steps": a["steps"], "act": a["act"], "cus": rng.choice([64, 128, 192, 256])}


# ------------------------------------------------------------------ inputs


def _gen(seed, what):
    return torch.Generator(device="cuda").manual_seed(1000 * seed + what)


def _weights(cfg, seed):
    """The flat fp32 parameter buffer (device), in the constructor's order."""
    schema = synth.weight_schema(cfg)
    w = torch.randn(synth.weight_count(cfg), generator=_gen(seed, 1), device="cuda") * 0.02
    off = 0
    for _, shape, kind in schema:
        n = math.prod(shape)
        if kind == synth.GAIN:
            w[off:off + n] += 1.0
        off += n
    return w


def _requests(cfg, batch, seed):
    g = _gen(seed, 2)
    d = {"pixels": torch.rand(batch, cfg.n_img, 3, cfg.img_hw, cfg.img_hw, generator=g, device="cuda"),
         "text": torch.randint(0, cfg.vocab, (batch, cfg.n_text), generator=g, device="cuda", dtype=torch.int32),
         "noise": torch.randn(batch, cfg.horizon, cfg.action_dim, generator=g, device="cuda"), "state": None}
    if cfg.head_kind == synth.HEAD_DIT:
        d["state"] = torch.randn(batch, cfg.state_dim, generator=g, device="cuda")
    return d


def _dtype(cfg):
    return torch.float32 if cfg.dtype == synth.DTYPE_F32 else torch.bfloat16


def _prefix(cfg, batch, seed):
    """A prefix state as the VLM stage leaves it (the element type's values, flat)."""
    g = _gen(seed, 3)
    if cfg.head_kind == synth.HEAD_JOINT:
        n = cfg.llm_layers * 2 * batch * cfg.n_kv * cfg.prefix_len * cfg.head_dim
        kv = torch.randn(n, generator=g, device="cuda") * (0.02 * math.sqrt(cfg.llm_d))
    else:
        n = batch * cfg.prefix_len * cfg.act_layers * 2 * cfg.act_d + batch * cfg.act_d
        kv = torch.randn(n, generator=g, device="cuda") * (0.02 * math.sqrt(cfg.act_d))
    return kv.to(_dtype(cfg))


def _model(cfg, seed):
    return vla.Model(cfg, _weights(cfg, seed).cpu().numpy())


_join = []


def _join_stream():
    if not _join:   # a serving loop's own stream, kept for the process
        _join.append(vla.nonblocking_stream(0))
    return _join[0]


def prepare(case, seed):
    if case["kind"] == "lockstep":
        v, a = _lockstep(case)
        return {"case": case, "vlm": prepare(v, seed), "act": prepare(a, seed), "stream": _join_stream()}
    cfg = _cfg(case)
    s = {"case": case, "cfg": cfg, "model": _model(cfg, seed)}
    s.update(_requests(cfg, case["batch"], seed))
    if case["kind"] == "action":
        s["kv"] = _prefix(cfg, case["batch"], seed)
    else:
        s["kv"] = s["model"].alloc_kv(case["batch"]).view(_dtype(cfg))
    s["actions"] = torch.empty_like(s["noise"])
    return s


# ------------------------------------------------------------------ one pass


def _hand_off(cfg, batch, kv):
    """The prefix state by layer (joint head) or its two parts (DiT head), as views."""
    if cfg.head_kind == synth.HEAD_JOINT:
        kv = kv.view(cfg.llm_layers, 2, batch, cfg.n_kv, cfg.prefix_len, cfg.head_dim)
        return {"layer%d" % l: kv[l] for l in range(cfg.llm_layers)}
    n = batch * cfg.prefix_len * cfg.act_layers * 2 * cfg.act_d
    return {"cross": kv[:n].view(batch, cfg.prefix_len, cfg.act_layers, 2, cfg.act_d),
            "state": kv[n:].view(batch, cfg.act_d)}


def run(s):
    c = s["case"]
    if c["kind"] == "lockstep":
        v, a = s["vlm"], s["act"]
        vla.step(v["model"], c["batch"], v["pixels"], v["text"], v["kv"], a["model"], c["act_batch"], a["kv"],
                 a["noise"], c["steps"], a["actions"], vlm_cu_count=c["cus"], join_stream=s["stream"])
        return {"vlm": _hand_off(v["cfg"], c["batch"], v["kv"]), "actions": a["actions"]}
    m, cfg, b = s["model"], s["cfg"], c["batch"]
    out = {}
    if c["kind"] != "action":
        m.prefill(b, s["pixels"], s["text"], s["kv"], state=s["state"])
        out["vlm"] = _hand_off(cfg, b, s["kv"])
    if c["kind"] != "vlm":
        m.denoise(b, s["kv"], s["noise"], c["steps"], s["actions"])
        out["actions"] = s["actions"]
    return out


# ------------------------------------------------------------------ work


def _vlm_work(cfg, b):
    es = 4 if cfg.dtype == synth.DTYPE_F32 else 2
    rows_i, rows, flops, wts = b * cfg.n_img * cfg.patch_tokens, b * cfg.prefix_len, 0, 0

    def mat(m, k, n):
        nonlocal flops, wts
        flops += 2 * m * k * n
        wts += k * n * es

    mat(rows_i, cfg.patch_dim, cfg.embed_d)
    d, f = cfg.vit_d, cfg.vit_mlp
    for _ in range(cfg.vit_layers):
        mat(rows_i, d, 3 * d), mat(rows_i, d, d), mat(rows_i, d, f), mat(rows_i, f, d)
        flops += 4 * rows_i * cfg.patch_tokens * d
    if cfg.vit_layers:
        mat(b * cfg.n_img_tokens, d * cfg.pix_shuffle ** 2, cfg.llm_d)
    hq, hk, d = cfg.n_q * cfg.head_dim, cfg.n_kv * cfg.head_dim, cfg.llm_d
    dit = cfg.head_kind == synth.HEAD_DIT
    for l in range(cfg.llm_layers):
        if not dit and l == cfg.llm_layers - 1:      # only this layer's keys and values are used
            mat(rows, d, 2 * hk)
            continue
        mat(rows, d, hq + 2 * hk), mat(rows, hq, d), mat(rows, d, 2 * cfg.llm_mlp), mat(rows, cfg.llm_mlp, d)
        flops += 4 * rows * cfg.prefix_len * hq
    if dit:
        mat(rows, d, cfg.act_d), mat(rows, cfg.act_d, 2 * cfg.act_layers * cfg.act_d)
        mat(b, cfg.state_dim, cfg.act_d)
        out = rows * cfg.act_layers * 2 * cfg.act_d * es
    else:
        out = cfg.llm_layers * 2 * rows * hk * es
    inp = b * (cfg.n_img * 3 * cfg.img_hw ** 2 * 4 + cfg.n_text * (4 + d * es))
    return wts + inp + out, flops


def _act_work(cfg, b, steps):
    es = 4 if cfg.dtype == synth.DTYPE_F32 else 2
    rows, d, f, flops, wts = b * cfg.n_tokens_act, cfg.act_d, cfg.act_mlp, 0, 0

    def mat(m, k, n):
        nonlocal flops, wts
        flops += 2 * m * k * n
        wts += k * n * es

    p, own = cfg.prefix_len, cfg.n_tokens_act
    mat(rows, cfg.action_dim, d)
    if cfg.head_kind == synth.HEAD_JOINT:
        hq, hk = cfg.n_q * cfg.head_dim, cfg.n_kv * cfg.head_dim
        mat(rows, d, d), mat(rows, d, cfg.action_dim)
        for _ in range(cfg.act_layers):
            mat(rows, d, hq + 2 * hk), mat(rows, hq, d), mat(rows, d, 2 * f), mat(rows, f, d)
            flops += 4 * rows * (p + own) * hq
        kv = cfg.llm_layers * 2 * b * p * hk * es
    else:
        mat(rows, d, cfg.action_dim)
        for _ in range(cfg.act_layers):
            mat(rows, d, 3 * d), mat(rows, d, d), mat(rows, d, d), mat(rows, d, d), mat(rows, d, f), mat(rows, f, d)
            flops += 4 * rows * (p + own) * d
        kv = b * p * cfg.act_layers * 2 * d * es
    # the weights and the prefix state once, however many steps read them
    return wts + kv + 2 * b * cfg.horizon * cfg.action_dim * 4, flops * steps


def work(case):
    if case["kind"] == "lockstep":
        v, a = (work(x) for x in _lockstep(case))
        return {k: v[k] + a[k] for k in v}
    cfg, b = _cfg(case), case["batch"]
    got = [(0, 0)]
    if case["kind"] != "action":
        got.append(_vlm_work(cfg, b))
    if case["kind"] != "vlm":
        got.append(_act_work(cfg, b, case["steps"]))
    return {"bytes": sum(x[0] for x in got), "flops": sum(x[1] for x in got)}


def tolerance(case):
    # about four times the distance from the 64-bit result that is measured over the range: fp32 throughout for the
    # small model (6e-7); the Euler loop over up to four bf16 action blocks, whose start, the noise, is exact (2e-3);
    # bf16 products through at most two ViT and three LLM blocks (6e-3). The largest of some million differences that
    # spread like rounding errors is about six times their root mean square.
    rel = {"request": 3e-6, "action": 8e-3}.get(case["kind"], 2.4e-2)
    return {"rel": rel, "max": 10 * rel}


# ------------------------------------------------------------------ 64-bit results


def _rms(x, g, eps):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps) * g


def _ln(x, eps):
    x = x - x.mean(-1, keepdim=True)
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + eps)


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _silu(x):
    return x / (1.0 + torch.exp(-x))


def _heads(x, n):       # [B, L, n * hd] -> [B, n, L, hd]
    b, l, d = x.shape
    return x.view(b, l, n, d // n).transpose(1, 2).contiguous()


def _attend(q, k, v):   # heads [B, n, L, hd]; grouped keys and values; -> [B, L, n * hd]
    b, n, l, hd = q.shape
    out = torch.empty(b, l, n, hd, dtype=q.dtype, device=q.device)
    for i in range(b):  # a request at a time bounds the score matrix
        for h in range(n):
            g = h * k.shape[1] // n
            s = q[i, h] @ k[i, g].t() / math.sqrt(hd)
            out[i, :, h] = torch.softmax(s, -1) @ v[i, g]
    return out.view(b, l, n * hd)


def _rope(x, pos, base):
    half = x.shape[-1] // 2
    a = pos[:, None] * base ** (-torch.arange(half, dtype=torch.float64, device=x.device) / half)
    c, s = torch.cos(a), torch.sin(a)
    lo, hi = x[..., :half], x[..., half:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _params(cfg, seed):
    w, off, out = _weights(cfg, seed), 0, {}
    w = w.to(_dtype(cfg))       # parameters are rounded to the model's type
    for name, shape, _ in synth.weight_schema(cfg):
        n = math.prod(shape)
        out[name] = w[off:off + n].view(shape)
        off += n
    return out


class _P:
    """Parameters in 64 bits, one at a time."""

    def __init__(self, cfg, seed):
        self.p = _params(cfg, seed)

    def __getitem__(self, name):
        return self.p[name].double()


def _vlm_exact(cfg, W, d, b):
    eps, base = cfg.norm_eps, cfg.rope_base
    g, p, t = cfg.patch_grid, cfg.patch, cfg.patch_tokens
    x = d["pixels"].double().view(b * cfg.n_img, 3, g, p, g, p).permute(0, 2, 4, 1, 3, 5).reshape(-1, t, 3 * p * p)
    x = x @ W["patch.w"] + W["patch.b"] + W["patch.pos"]
    for l in range(cfg.vit_layers):
        n = "vit.%d." % l
        z = _ln(x, eps) * W[n + "ln1.g"] + W[n + "ln1.b"]
        q, k, v = (_heads(z @ W[n + "w" + i] + W[n + "b" + i], cfg.vit_heads) for i in "qkv")
        x = x + _attend(q, k, v) @ W[n + "wo"] + W[n + "bo"]
        z = _ln(x, eps) * W[n + "ln2.g"] + W[n + "ln2.b"]
        x = x + _gelu(z @ W[n + "w1"] + W[n + "b1"]) @ W[n + "w2"] + W[n + "b2"]
    if cfg.vit_layers:
        x = _ln(x, eps) * W["vit.lnf.g"] + W["vit.lnf.b"]
        s = cfg.pix_shuffle
        x = x.view(-1, g // s, s, g // s, s, cfg.vit_d).permute(0, 1, 3, 2, 4, 5).reshape(
            b * cfg.n_img, t // s ** 2, s * s * cfg.vit_d)
        x = x @ W["vit.proj.w"] + W["vit.proj.b"]
    h = torch.cat([x.reshape(b, -1, cfg.llm_d), W["embed"][d["text"].long()]], 1)
    pos = torch.arange(h.shape[1], dtype=torch.float64, device=h.device)
    dit, out = cfg.head_kind == synth.HEAD_DIT, {}
    for l in range(cfg.llm_layers):
        n = "llm.%d." % l
        z = _rms(h, W[n + "ln1.g"], eps)
        q = _rope(_heads(z @ W[n + "wq"], cfg.n_q), pos, base)
        k, v = _rope(_heads(z @ W[n + "wk"], cfg.n_kv), pos, base), _heads(z @ W[n + "wv"], cfg.n_kv)
        if not dit:
            out["layer%d" % l] = torch.stack([k, v])
            if l == cfg.llm_layers - 1:
                return out
        h = h + _attend(q, k, v) @ W[n + "wo"]
        z = _rms(h, W[n + "ln2.g"], eps)
        h = h + (_gelu(z @ W[n + "wg"]) * (z @ W[n + "wu"])) @ W[n + "wd"]
    f = _rms(h, W["llm.lnf.g"], eps) @ W["vp.w"] + W["vp.b"]
    kv = [torch.stack([f @ W["xkv.%d.w%s" % (l, i)] + W["xkv.%d.b%s" % (l, i)] for i in "kv"], 2)
          for l in range(cfg.act_layers)]
    return {"cross": torch.stack(kv, 2), "state": d["state"].double() @ W["state.w"] + W["state.b"]}


def _sinusoid(t, dim):
    a = 1000.0 * t * 10000.0 ** (-torch.arange(dim // 2, dtype=torch.float64, device="cuda") / (dim // 2))
    return torch.cat([torch.sin(a), torch.cos(a)])


def _joint_velocity(cfg, W, pre, x, t):
    eps, base, p = cfg.norm_eps, cfg.rope_base, cfg.prefix_len
    e = x @ W["act.in.w"] + W["act.in.b"]
    e = _silu(e @ W["act.t1a.w"] + _sinusoid(t, cfg.tdim) @ W["act.t1t.w"] + W["act.t1.b"])
    h = e @ W["act.t2.w"] + W["act.t2.b"]
    pos = p + torch.arange(cfg.horizon, dtype=torch.float64, device=h.device)
    for l in range(cfg.act_layers):
        n = "act.%d." % l
        z = _rms(h, W[n + "ln1.g"], eps)
        q = _rope(_heads(z @ W[n + "wq"], cfg.n_q), pos, base)
        k, v = _rope(_heads(z @ W[n + "wk"], cfg.n_kv), pos, base), _heads(z @ W[n + "wv"], cfg.n_kv)
        k, v = (torch.cat([pre["layer%d" % l][i].double(), y], 2) for i, y in enumerate((k, v)))
        h = h + _attend(q, k, v) @ W[n + "wo"]
        z = _rms(h, W[n + "ln2.g"], eps)
        h = h + (_gelu(z @ W[n + "wg"]) * (z @ W[n + "wu"])) @ W[n + "wd"]
    return _rms(h, W["act.lnf.g"], eps) @ W["act.out.w"] + W["act.out.b"]


def _dit_velocity(cfg, W, pre, x, t):
    eps, nh = cfg.norm_eps, cfg.act_heads
    c = _silu(_sinusoid(t, cfg.tdim) @ W["dit.t1.w"] + W["dit.t1.b"]) @ W["dit.t2.w"] + W["dit.t2.b"]
    sc = _silu(c)
    X = torch.cat([pre["state"].double()[:, None], x @ W["dit.ain.w"] + W["dit.ain.b"]], 1) + W["dit.pos"]
    for l in range(cfg.act_layers):
        n = "dit.%d." % l
        sh1, s1, g1, sh2, s2, g2 = (sc @ W[n + "mod.w"] + W[n + "mod.b"]).chunk(6)
        z = _ln(X, eps) * (1 + s1) + sh1
        q, k, v = (_heads(z @ W[n + "w" + i] + W[n + "b" + i], nh) for i in "qkv")
        X = X + g1 * (_attend(q, k, v) @ W[n + "wo"] + W[n + "bo"])
        q = _heads(_ln(X, eps) @ W[n + "cq.w"] + W[n + "cq.b"], nh)
        kc, vc = (_heads(pre["cross"][:, :, l, i].double(), nh) for i in (0, 1))
        X = X + _attend(q, kc, vc) @ W[n + "co.w"] + W[n + "co.b"]
        z = _ln(X, eps) * (1 + s2) + sh2
        X = X + g2 * (_gelu(z @ W[n + "w1"] + W[n + "b1"]) @ W[n + "w2"] + W[n + "b2"])
    sh, s = (sc @ W["dit.modf.w"] + W["dit.modf.b"]).chunk(2)
    return (_ln(X, eps) * (1 + s) + sh)[:, 1:] @ W["dit.out.w"] + W["dit.out.b"]


def exact(case, seed):
    if case["kind"] == "lockstep":
        v, a = (exact(x, seed) for x in _lockstep(case))
        return {**v, **a}
    cfg, b, out = _cfg(case), case["batch"], {}
    W, d = _P(cfg, seed), _requests(cfg, case["batch"], seed)
    if case["kind"] == "action":
        pre = _hand_off(cfg, b, _prefix(cfg, b, seed))
    else:
        pre = out["vlm"] = _vlm_exact(cfg, W, d, b)
    if case["kind"] != "vlm":
        x, n = d["noise"].double(), case["steps"]
        velocity = _joint_velocity if cfg.head_kind == synth.HEAD_JOINT else _dit_velocity
        for k in range(n):
            x = x - velocity(cfg, W, pre, x, 1.0 - k / n) / n
        out["actions"] = x
    return out
