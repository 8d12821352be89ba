"""The calls that a robot-policy program makes of this library, as timed cases.

A pi-family policy turns an observation into an action chunk in three phases,
each one entry point: the vision tower (``VisionTower.encode``), the language
prefix (``PrefixLM.prefill``) and the action expert's denoising loop
(``Expert.denoise``).  A robot calls them for one observation at a time and
waits; a rollout or serving program calls them for many requests with ragged
prefixes.  Both kinds are listed, for every expert variant and weight format.

A program loads its checkpoint once and keeps the handle, so the handle of a
shape is made once (weights from a fixed seed) and kept while the same shape is
asked for; what changes from call to call (prefix, noise, state, embeddings,
patches, prefix lengths) is made from the case's seed.
"""
from __future__ import annotations

import math
import types

import numpy as np
import torch

import paper_2608_03682_amd as px

INIT_STD = 0.02                     # weights ~ N(0, 0.02), inputs ~ N(0, 1)
WEIGHT_SEED = 20260801
EPS = 1e-6
PERIODS = (4e-3, 4.0)               # sinusoidal timestep embedding, shortest and longest period
ROPE_BASE = 10000.0
TRUNK = ("wq", "wk", "wv", "wo", "w_gate", "w_up", "w_down", "mlp_w1", "mlp_w2")

# The widths of each model.  tiny: the small fp32 expert; pi0 / pi05 / dit: the
# three action experts; lm: the Gemma-class language part; tower: the
# SigLIP-class vision transformer.
MODELS = {
    "tiny": dict(variant="pi0", d=256, nq=4, nkv=1, D=64, F=1024, rope=False, token=False, time_dim=256),
    "pi0": dict(variant="pi0", d=1024, nq=8, nkv=1, D=256, F=4096, rope=True, token=True, time_dim=1024),
    "pi05": dict(variant="pi05", d=1024, nq=8, nkv=1, D=256, F=4096, rope=True, token=False, time_dim=1024),
    "dit": dict(variant="dit", d=1536, nq=12, nkv=12, D=128, F=6144, rope=False, token=True, time_dim=256,
                d_feat=2048),
    "lm": dict(variant="prefix_lm", d=2048, nq=8, nkv=1, D=256, F=16384, rope=True, token=False, time_dim=0),
    "tower": dict(variant="vision", d=1024, nq=16, nkv=16, D=64, F=4096, rope=False, token=False, time_dim=0,
                  patch_dim=768, d_out=2048),
}


def expert(name, model, weights, layers, steps, batch, prefix, prefix_min, horizon=50, actions=32):
    return {"name": name, "model": model, "weights": weights, "layers": layers, "steps": steps, "batch": batch,
            "prefix": prefix, "prefix_min": prefix_min, "horizon": horizon, "actions": actions}


def listed():
    return [
        # the smallest call: a two-layer fp32 expert, launches and latency only
        expert("tiny_fp32_b1", "tiny", "f32", 2, 4, 1, 64, 64, horizon=16, actions=7),
        # one robot, one observation: the whole pi0 chunk, 10 Euler steps over
        # 3 x 256 image tokens and 48 of text
        expert("pi0_bf16_b1", "pi0", "bf16", 18, 10, 1, 816, 816),
        # the same for pi0.5 (adaRMSNorm; 200 text and state tokens)
        expert("pi05_bf16_b1", "pi05", "bf16", 18, 10, 1, 968, 968),
        # the DiT action head: 16 actions, 300 feature tokens, 4 steps
        expert("dit_bf16_b1", "dit", "bf16", 16, 4, 1, 300, 300, horizon=16),
        # pi0 with 4-bit weights on one robot
        expert("pi0_fp4_b1", "pi0", "fp4", 18, 10, 1, 816, 816),
        # a few robots behind one GPU: ragged prefixes, a batch between the two extremes
        expert("pi0_bf16_b8", "pi0", "bf16", 18, 10, 8, 1000, 600),
        # pi0.5 serving at the batch of the phase analysis (32 requests); six of
        # its 18 layers, which are alike
        expert("pi05_bf16_b32", "pi05", "bf16", 6, 10, 32, 1000, 600),
        # cloud rollouts: 64 requests, fp8 weights, ragged prefixes
        expert("pi0_fp8_b64", "pi0", "fp8", 18, 10, 64, 1000, 600),
        # the language prefix of one observation; four of the 18 layers
        {"name": "lm_bf16_b1", "model": "lm", "weights": "bf16", "layers": 4, "batch": 1, "prefix": 816,
         "prefix_min": 816},
        # the language prefix of four ragged requests
        {"name": "lm_bf16_b4", "model": "lm", "weights": "bf16", "layers": 4, "batch": 4, "prefix": 1000,
         "prefix_min": 600},
        # the vision tower over one observation's three camera images, whole
        {"name": "tower_bf16_b1", "model": "tower", "weights": "bf16", "layers": 24, "batch": 1, "images": 3,
         "patches": 256},
        # the vision tower at 32 observations; six of the 24 blocks
        {"name": "tower_bf16_b32", "model": "tower", "weights": "bf16", "layers": 6, "batch": 32, "images": 3,
         "patches": 256},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    model = rng.choice(["tiny", "pi0", "pi0", "pi0", "pi05", "pi05", "dit", "lm", "tower"])
    if model == "tower":
        images = rng.randint(1, 3)
        return {"model": model, "weights": rng.choice(["bf16", "bf16", "fp8"]), "layers": rng.randint(2, 6),
                "batch": _log_int(rng, 1, 32), "images": images, "patches": rng.randint(60, 256)}
    if model == "lm":
        cap = rng.randint(150, 1000)
        return {"model": model, "weights": rng.choice(["bf16", "bf16", "fp8"]), "layers": rng.randint(2, 4),
                "batch": rng.randint(1, 4), "prefix": cap, "prefix_min": rng.randint(cap // 2, cap)}
    if model == "tiny":
        cap = rng.randint(16, 128)
        return dict(model=model, weights="f32", layers=rng.randint(1, 3), steps=rng.randint(2, 8),
                    batch=rng.randint(1, 4), prefix=cap, prefix_min=rng.randint(cap // 2, cap),
                    horizon=rng.randint(8, 32), actions=rng.choice([7, 14, 32]))
    if model == "dit":
        cap = rng.randint(50, 400)
        return dict(model=model, weights="bf16", layers=2 * rng.randint(1, 4), steps=rng.randint(2, 8),
                    batch=_log_int(rng, 1, 16), prefix=cap, prefix_min=rng.randint(cap // 2, cap),
                    horizon=rng.randint(8, 32), actions=rng.choice([7, 14, 32]))
    weights = rng.choice(["bf16", "fp8", "fp4"]) if model == "pi0" else "bf16"
    cap = rng.randint(200, 1000)
    return dict(model=model, weights=weights, layers=rng.randint(2, 6), steps=rng.randint(2, 10),
                batch=_log_int(rng, 1, 16 if weights == "fp4" else 64 if weights == "fp8" else 32), prefix=cap,
                prefix_min=rng.randint(cap // 2, cap), horizon=rng.randint(10, 60), actions=rng.choice([7, 14, 24, 32]))


# ----------------------------------------------------------------------------
# weights
# ----------------------------------------------------------------------------

def _specs(case):
    """name -> (rows, columns), every tensor the handle of this case takes."""
    m = MODELS[case["model"]]
    d, F, v, A, L = m["d"], m["F"], m["variant"], case.get("actions", 0), case["layers"]
    qd, kd = m["nq"] * m["D"], m["nkv"] * m["D"]
    s = {}
    if v == "vision":
        s.update(patch_w=(m["patch_dim"], d), patch_b=(1, d), pos_emb=(case["patches"], d), post_ln_w=(1, d),
                 post_ln_b=(1, d), proj_w=(d, m["d_out"]), proj_b=(1, m["d_out"]))
    elif v != "prefix_lm":
        s.update(in_w=(A, d), in_b=(1, d), out_w=(d, A), out_b=(1, A))
        if m["token"]:
            s.update(state_w=(A, d), state_b=(1, d))
        if v == "pi0":
            s.update(time_w1=(d + m["time_dim"], d), time_b1=(1, d), time_w2=(d, d), time_b2=(1, d), final_norm=(1, d))
        else:
            s.update(cond_w1=(m["time_dim"], d), cond_b1=(1, d), cond_w2=(d, d), cond_b2=(1, d))
            fin = "final_mod" if v == "pi05" else "final_ada"
            s.update({fin + "_w": (d, 2 * d), fin + "_b": (1, 2 * d)})
        if v == "dit":
            s["pos_emb"] = (case["horizon"], d)
    for l in range(L):
        kin = m["d_feat"] if v == "dit" and l % 2 == 0 else d
        t = dict(wq=(d, qd), wk=(kin, kd), wv=(kin, kd), wo=(qd, d))
        if v == "vision":
            t.update(ln1_w=(1, d), ln1_b=(1, d), ln2_w=(1, d), ln2_b=(1, d), bq=(1, d), bk=(1, d), bv=(1, d), bo=(1, d))
        if v in ("vision", "dit"):
            t.update(mlp_w1=(d, F), mlp_b1=(1, F), mlp_w2=(F, d), mlp_b2=(1, d))
        else:
            t.update(w_gate=(d, F), w_up=(d, F), w_down=(F, d))
        if v in ("pi0", "prefix_lm"):
            t.update(attn_norm=(1, d), mlp_norm=(1, d))
        elif v == "pi05":
            t.update(attn_mod_w=(d, 2 * d), attn_mod_b=(1, 2 * d), mlp_mod_w=(d, 2 * d), mlp_mod_b=(1, 2 * d))
        elif v == "dit":
            t.update(ada_w=(d, 6 * d), ada_b=(1, 6 * d))
        if v == "prefix_lm" and l + 1 == L:       # the last layer ends with its keys and values
            t = {k: t[k] for k in ("attn_norm", "wq", "wk", "wv")}
        s.update({f"layers.{l}.{k}": x for k, x in t.items()})
    return s


def _format(case, name):
    w = case["weights"]
    if w in ("fp8", "fp4"):
        return w if name.startswith("layers.") and name.rsplit(".", 1)[-1] in TRUNK else "bf16"
    return w


def _weights(case, stored):
    """Each tensor of the case's checkpoint in turn: as the library takes it
    (stored) or as the 64-bit values that this storage holds."""
    gen = torch.Generator(device="cuda").manual_seed(WEIGHT_SEED)
    grid = torch.tensor([0, 0.5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device="cuda")
    for name, shape in sorted(_specs(case).items()):
        x = torch.randn(shape, generator=gen, device="cuda") * INIT_STD
        fmt, scale = _format(case, name), None
        if fmt == "f32":
            data, value = x, x.double()
        elif fmt == "bf16":
            data = x.bfloat16()
            value = data.double()
            data = data.view(torch.int16)
        elif fmt == "fp8":                        # one scale per output column
            scale = x.abs().amax(0) / 448
            data = (x / scale).to(torch.float8_e4m3fn)
            value = data.double() * scale.double()
            data = data.view(torch.uint8)
        else:                                     # e2m1, a power-of-two scale per 32 rows and column
            g = x.double().view(-1, 32, shape[1])
            scale = torch.exp2(torch.ceil(torch.log2(g.abs().amax(1) / 6)))
            g = g / scale[:, None]
            code = torch.bucketize(g.abs(), (grid[1:] + grid[:-1]) / 2)
            value = (grid[code] * g.sign() * scale[:, None]).view(shape)
            code = (code + 8 * (g < 0)).to(torch.uint8).view(shape)
            data, scale = code[:, 0::2] | (code[:, 1::2] << 4), scale.float()
        if not stored:
            yield name, value
            continue
        data = data.cpu().numpy()
        if fmt == "bf16":
            data = data.view(np.uint16)
        yield name, types.SimpleNamespace(dtype=fmt, data=data, scale=None if scale is None else scale.cpu().numpy())


_kept = {}                                        # the handle of the shape asked for last


def _handle(case):
    key = repr(sorted((k, x) for k, x in case.items() if k not in ("name", "prefix_min")))
    if key not in _kept:
        _kept.clear()
        m = MODELS[case["model"]]
        v = m["variant"]
        cfg = types.SimpleNamespace(
            variant=v, n_layers=case["layers"], d_model=m["d"], n_q_heads=m["nq"], n_kv_heads=m["nkv"],
            head_dim=m["D"], d_mlp=m["F"], horizon=case.get("horizon", 0), action_dim=case.get("actions", 0),
            n_steps=case.get("steps", 0), prefix_cap=case.get("prefix", 0), batch=case["batch"], state_token=m["token"],
            rope=m["rope"], weight_dtype=case["weights"], kv_dtype="f32" if case["weights"] == "f32" else "bf16",
            d_feat=m.get("d_feat", 0), time_dim=m["time_dim"], rms_eps=EPS, sin_min_period=PERIODS[0],
            sin_max_period=PERIODS[1], rope_base=ROPE_BASE, n_images=case.get("images", 0),
            n_patches=case.get("patches", 0), patch_dim=m.get("patch_dim", 0), d_out=m.get("d_out", 0))
        make = {"prefix_lm": px.PrefixLM, "vision": px.VisionTower}.get(v, px.Expert)
        _kept[key] = make(cfg, dict(_weights(case, stored=True)))
    return _kept[key]


# ----------------------------------------------------------------------------
# the calls
# ----------------------------------------------------------------------------

def _inputs(case, seed):
    m = MODELS[case["model"]]
    gen = torch.Generator(device="cuda").manual_seed(seed)
    B, P = case["batch"], case.get("prefix", 0)
    kv = torch.float32 if case["weights"] == "f32" else torch.bfloat16
    s = types.SimpleNamespace(model=case["model"])

    def randn(*shape, dtype=torch.float32):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dtype)

    if m["variant"] == "vision":
        s.patches = randn(B, case["images"], case["patches"], m["patch_dim"])
        return s
    s.prefix_len = np.random.default_rng(seed).integers(case["prefix_min"], P + 1, size=B).astype(np.int32)
    if m["variant"] == "prefix_lm":
        s.embeds = randn(B, P, m["d"])
        return s
    shape = (B, P, m["d_feat"]) if m["variant"] == "dit" else (case["layers"], 2, B, P, m["nkv"] * m["D"])
    s.prefix = randn(*shape, dtype=kv)
    s.noise = randn(B, case["horizon"], case["actions"])
    s.state = randn(B, case["actions"]) if m["token"] else None
    s.timesteps = (1.0 - np.arange(case["steps"] + 1) / case["steps"]).astype(np.float32)
    return s


def prepare(case, seed):
    m = MODELS[case["model"]]
    s = _inputs(case, seed)
    s.handle = _handle(case)
    B = case["batch"]
    if m["variant"] == "vision":
        s.out = torch.empty((B, case["images"] * case["patches"], m["d_out"]), device="cuda")
    elif m["variant"] == "prefix_lm":
        s.out = torch.empty((case["layers"], 2, B, case["prefix"], m["nkv"] * m["D"]), device="cuda",
                            dtype=torch.bfloat16)
    else:
        s.out = torch.empty_like(s.noise)
        s.handle.prepare(B, case["steps"])
    return s


def run(s):
    if s.model == "tower":
        return s.handle.encode(s.patches, out=s.out)
    if s.model == "lm":
        return s.handle.prefill(s.embeds, s.prefix_len, out=s.out)
    return s.handle.denoise(s.prefix, s.prefix_len, s.noise, s.timesteps, s.state, out=s.out)


def work(case):
    """Weights and inputs read once, outputs written once; the products of
    every projection and of attention over the mean prefix."""
    m = MODELS[case["model"]]
    v, B, L, steps = m["variant"], case["batch"], case["layers"], case.get("steps", 1)
    size = {"f32": 4, "bf16": 2, "fp8": 1, "fp4": 0.5 + 1 / 32}
    act = 4 if case["weights"] == "f32" else 2
    specs = _specs(case)
    nbytes = sum(r * c * size[_format(case, k)] for k, (r, c) in specs.items())
    trunk = [(k, r * c) for k, (r, c) in specs.items() if k.startswith("layers.") and k.rsplit(".", 1)[-1] in TRUNK]
    P = (case["prefix"] + case["prefix_min"]) / 2 if "prefix" in case else 0
    qd, kd = m["nq"] * m["D"], m["nkv"] * m["D"]
    if v == "vision":
        I, N = case["images"], case["patches"]
        rows = B * I * N
        flops = 2 * rows * (sum(n for _, n in trunk) + m["patch_dim"] * m["d"] + m["d"] * m["d_out"])
        flops += L * 4 * rows * N * qd
        return {"bytes": nbytes + 4 * rows * (m["patch_dim"] + m["d_out"]), "flops": flops}
    if v == "prefix_lm":
        flops = 2 * B * P * sum(n for _, n in trunk) + (L - 1) * 4 * B * P * P * qd
        return {"bytes": nbytes + B * P * 4 * m["d"] + L * 2 * B * case["prefix"] * kd * act, "flops": flops}
    H, A = case["horizon"], case["actions"]
    M = H + (1 if m["token"] else 0)
    io = 4 * B * (2 * H * A + (A if m["token"] else 0))
    if v == "dit":
        cross = [n for k, n in trunk if k.rsplit(".", 1)[-1] in ("wk", "wv") and int(k.split(".")[1]) % 2 == 0]
        flops = 2 * B * P * sum(cross) + steps * 2 * B * M * (sum(n for _, n in trunk) - sum(cross))
        flops += steps * 4 * B * M * qd * (P * len(cross) / 2 + M * (L - len(cross) / 2))
        return {"bytes": nbytes + io + B * P * m["d_feat"] * act, "flops": flops}
    flops = steps * (2 * B * M * sum(n for _, n in trunk) + L * 4 * B * M * (P + M) * qd)
    flops += steps * 2 * B * H * A * m["d"] * 2
    return {"bytes": nbytes + io + L * 2 * B * P * kd * act, "flops": flops}


# About four times the relative error against 64 bits that the whole models
# show: 32-bit throughout 2.2e-6; bf16 operands with 32-bit sums 2.9e-3 (pi0),
# 1.3e-3 (pi0.5 and DiT, whose output moves less against the noise), 4.2e-3
# (the language prefix and the tower, whose outputs are the last layer's own).
def tolerance(case):
    if case["weights"] == "f32":
        return {"rel": 1e-5}
    return {"rel": {"pi0": 1.2e-2, "pi05": 5e-3, "dit": 5e-3, "lm": 1.5e-2, "tower": 1.6e-2}[case["model"]]}


# ----------------------------------------------------------------------------
# the same in 64 bits
# ----------------------------------------------------------------------------

def _rms(h):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + EPS)


def _layer_norm(h):
    c = h - h.mean(-1, keepdim=True)
    return c / torch.sqrt((c * c).mean(-1, keepdim=True) + EPS)


def _gelu(z):
    return 0.5 * z * (1 + torch.tanh(math.sqrt(2 / math.pi) * (z + 0.044715 * z ** 3)))


def _swish(z):
    return z * torch.sigmoid(z)


def _rope(x, pos):
    """x [rows, heads, D], pos [rows]: pairs (i, i + D/2) turned by pos * base^(-2i/D)."""
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * ROPE_BASE ** (-torch.arange(half, device="cuda", dtype=torch.float64) / half)
    c, s = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, b = x[..., :half], x[..., half:]
    return torch.cat([a * c - b * s, b * c + a * s], -1)


def _attend(q, k, v, mask=None):
    """q [M, nq, D], k, v [N, nkv, D]; mask [M, N], True where a key counts."""
    M, nq, D = q.shape
    nkv = k.shape[1]
    G = nq // nkv
    out = torch.empty_like(q)
    for h in range(nkv):
        s = q[:, h * G:(h + 1) * G].reshape(M * G, D) @ k[:, h].T / math.sqrt(D)
        if mask is not None:
            s = s.masked_fill(~mask.repeat_interleave(G, 0), -math.inf)
        out[:, h * G:(h + 1) * G] = (torch.softmax(s, -1) @ v[:, h]).view(M, G, D)
    return out


def _tau(t, n):
    i = torch.arange(n // 2, device="cuda", dtype=torch.float64) / (n // 2 - 1)
    ang = 2 * math.pi * t / (PERIODS[0] * (PERIODS[1] / PERIODS[0]) ** i)
    return torch.cat([torch.sin(ang), torch.cos(ang)])


def exact(case, seed):
    m, s, W = MODELS[case["model"]], _inputs(case, seed), dict(_weights(case, stored=False))
    run64 = {"vision": _exact_tower, "prefix_lm": _exact_lm}.get(m["variant"], _exact_expert)
    return run64(case, m, s, W)


def _exact_tower(case, m, s, W):
    B, I, N = case["batch"], case["images"], case["patches"]
    nq, D = m["nq"], m["D"]
    h = s.patches.double().view(B * I, N, -1) @ W["patch_w"] + W["patch_b"] + W["pos_emb"]
    for l in range(case["layers"]):
        w = {k.split(".")[2]: x for k, x in W.items() if k.startswith(f"layers.{l}.")}
        a = _layer_norm(h) * (1 + w["ln1_w"]) + w["ln1_b"]
        q, k, v = ((a @ w["w" + c] + w["b" + c]).view(B * I, N, nq, D) for c in "qkv")
        o = torch.stack([_attend(q[i], k[i], v[i]) for i in range(B * I)]).view(B * I, N, nq * D)
        h = h + o @ w["wo"] + w["bo"]
        a = _layer_norm(h) * (1 + w["ln2_w"]) + w["ln2_b"]
        h = h + _gelu(a @ w["mlp_w1"] + w["mlp_b1"]) @ w["mlp_w2"] + w["mlp_b2"]
    z = _layer_norm(h) * (1 + W["post_ln_w"]) + W["post_ln_b"]
    return (z @ W["proj_w"] + W["proj_b"]).view(B, I * N, -1)


def _exact_lm(case, m, s, W):
    B, P, L = case["batch"], case["prefix"], case["layers"]
    nq, nkv, D = m["nq"], m["nkv"], m["D"]
    out = torch.zeros((L, 2, B, P, nkv * D), device="cuda", dtype=torch.float64)
    for b in range(B):
        n = int(s.prefix_len[b])
        h, pos = s.embeds[b, :n].double(), torch.arange(n, device="cuda")
        for l in range(L):
            w = {k.split(".")[2]: x for k, x in W.items() if k.startswith(f"layers.{l}.")}
            a = _rms(h) * (1 + w["attn_norm"])
            k, v = _rope((a @ w["wk"]).view(n, nkv, D), pos), (a @ w["wv"]).view(n, nkv, D)
            out[l, 0, b, :n], out[l, 1, b, :n] = k.view(n, -1), v.view(n, -1)
            if l + 1 == L:
                break
            q = _rope((a @ w["wq"]).view(n, nq, D), pos)
            h = h + _attend(q, k, v).view(n, nq * D) @ w["wo"]
            a = _rms(h) * (1 + w["mlp_norm"])
            h = h + (_gelu(a @ w["w_gate"]) * (a @ w["w_up"])) @ w["w_down"]
    return out


def _exact_expert(case, m, s, W):
    v, B, H, L, d = m["variant"], case["batch"], case["horizon"], case["layers"], m["d"]
    nq, nkv, D, off = m["nq"], m["nkv"], m["D"], 1 if m["token"] else 0
    M = H + off
    layers = [{k.split(".")[2]: x for k, x in W.items() if k.startswith(f"layers.{l}.")} for l in range(L)]
    plen = [int(p) for p in s.prefix_len]
    pos = torch.cat([p + torch.arange(M, device="cuda") for p in plen])
    token = (s.state.double() @ W["state_w"] + W["state_b"])[:, None] if off else None
    # the keys and values that stay fixed over the steps
    fixed = {}
    for l in range(L):
        for b in range(B):
            if v != "dit":
                fixed[l, b] = [s.prefix[l, j, b, :plen[b]].double().view(-1, nkv, D) for j in (0, 1)]
            elif l % 2 == 0:
                f = s.prefix[b, :plen[b]].double()
                fixed[l, b] = [(f @ layers[l][c]).view(-1, nkv, D) for c in ("wk", "wv")]
    masks = [None] * B
    if v == "pi0" and off:                        # the state token sees the prefix and itself
        masks = [torch.ones((M, p + M), dtype=torch.bool, device="cuda") for p in plen]
        for x, p in zip(masks, plen):
            x[0, p + 1:] = False

    def velocity(x, t):
        a = x @ W["in_w"] + W["in_b"]
        tau = _tau(t, m["time_dim"])
        if v == "pi0":
            z = torch.cat([a, tau.expand(B, H, -1)], -1)
            a = _swish(z @ W["time_w1"] + W["time_b1"]) @ W["time_w2"] + W["time_b2"]
        else:
            c = _swish(_swish(tau @ W["cond_w1"] + W["cond_b1"]) @ W["cond_w2"] + W["cond_b2"])
        if v == "dit":
            a = a + W["pos_emb"]
        h = (torch.cat([token, a], 1) if off else a).reshape(B * M, d)

        def norm(h, w, site):
            if v == "pi0":
                return _rms(h) * (1 + w[site + "_norm"])
            mod = c @ w[site + "_mod_w"] + w[site + "_mod_b"]
            return _rms(h) * (1 + mod[:, :d]) + mod[:, d:]

        for l, w in enumerate(layers):
            if v == "dit":
                sh1, sc1, g1, sh2, sc2, g2 = (c @ w["ada_w"] + w["ada_b"])[0].split(d)
                a = _layer_norm(h) * (1 + sc1) + sh1
            else:
                g1 = g2 = 1.0
                a = norm(h, w, "attn")
            q = (a @ w["wq"]).view(B * M, nq, D)
            cross = v == "dit" and l % 2 == 0
            if not cross:
                k, val = (a @ w["wk"]).view(B * M, nkv, D), (a @ w["wv"]).view(B * M, nkv, D)
            if m["rope"]:
                q, k = _rope(q, pos), _rope(k, pos)
            o = torch.empty_like(q)
            for b in range(B):
                r = slice(b * M, (b + 1) * M)
                kv = fixed[l, b] if cross else [k[r], val[r]] if v == "dit" else [
                    torch.cat([fixed[l, b][0], k[r]]), torch.cat([fixed[l, b][1], val[r]])]
                o[r] = _attend(q[r], kv[0], kv[1], masks[b])
            h = h + g1 * (o.view(B * M, nq * D) @ w["wo"])
            if v == "dit":
                a = _layer_norm(h) * (1 + sc2) + sh2
                h = h + g2 * (_gelu(a @ w["mlp_w1"] + w["mlp_b1"]) @ w["mlp_w2"] + w["mlp_b2"])
            else:
                a = norm(h, w, "mlp")
                h = h + (_gelu(a @ w["w_gate"]) * (a @ w["w_up"])) @ w["w_down"]
        h = h.view(B, M, d)[:, off:]
        if v == "pi0":
            h = _rms(h) * (1 + W["final_norm"])
        elif v == "pi05":
            mod = (c @ W["final_mod_w"] + W["final_mod_b"])[0]
            h = _rms(h) * (1 + mod[:d]) + mod[d:]
        else:
            shift, scale = (c @ W["final_ada_w"] + W["final_ada_b"])[0].split(d)
            h = _layer_norm(h) * (1 + scale) + shift
        return h @ W["out_w"] + W["out_b"]

    x, ts = s.noise.double(), [float(t) for t in s.timesteps]
    for t, u in zip(ts, ts[1:]):
        x = x + (u - t) * velocity(x, t)
    return x
