"""The calls that a program built on this library makes, as cases to be timed.

A case names an entry point (``call``), a model shape and the options of the call:

``step``     ``Buffer.step``: one control step of rolling denoising (what a control loop calls at
             every tick), with ``refresh`` > 0 after publishing the contexts whose turn it is;
``state``    ``Buffer.step_state``: the same with relative action dimensions;
``full``     ``Buffer.full_denoise``: a whole chunk from noise, ``euler`` expert passes;
``train``    ``Buffer.train_loss``: the streaming-aligned objective's forward pass and loss, the
             predicted velocities returned too;
``encode``   ``Buffer.fop_encode``: the fast-observation encoder.

Weights are N(0, 1/sqrt(fan_in)) with +1 on the residual gates' biases and adapter gates of 1, so
that every sub-block moves the outputs; contexts, tokens and noise are N(0, 1).
"""

import math
import types

import numpy as np
import torch

from paper_2609_34170_amd import ravel

DEV = "cuda:0"

# The model families of the workloads: two layers in 32 bits, the small bf16 expert, the pi0.5-style
# expert and the large expert (heads as query/key-value x dim).
FAMILIES = {
    "tiny": dict(width=128, nq=4, nkv=4, hd=32, mlp=512, horizon=8, action_dim=7, prefix=32, fop=4, obs=32),
    "small": dict(width=512, nq=8, nkv=8, hd=64, mlp=2048, horizon=16, action_dim=14, prefix=256, fop=8, obs=64),
    "pi": dict(width=1024, nq=8, nkv=1, hd=256, mlp=4096, horizon=50, action_dim=32, prefix=816, fop=16, obs=256),
    "large": dict(width=2048, nq=16, nkv=4, hd=128, mlp=8192, horizon=100, action_dim=32, prefix=2048, fop=32,
                  obs=512),
}


def _case(family, call, layers, batch, **kw):
    c = dict(call=call, family=family, layers=layers, batch=batch, dtype="bf16", offset="mlp", rope=0.0, ages=1,
             refresh=0, euler=0)
    c.update(FAMILIES[family])
    c.update(kw)
    return c


def listed():
    cases = {
        # the smallest 32-bit expert, one robot: a chain of small launches
        "step_tiny_f32_b1": _case("tiny", "step", 2, 1, dtype="f32"),
        # the small bf16 expert, one robot
        "step_small_b1": _case("small", "step", 6, 1),
        # the pi0.5-style expert at its full depth, one robot: the latency of a control loop
        "step_pi_b1": _case("pi", "step", 18, 1, ages=4),
        # a few robots or simulator instances on one GPU
        "step_pi_b4": _case("pi", "step", 6, 4, ages=4),
        # a fleet of 64 environments whose contexts are refreshed in turn, every fifth step
        "step_pi_b64": _case("pi", "step", 6, 64, refresh=5),
        # the large expert for one robot: 100 slots, weights read for few rows
        "step_large_b1": _case("large", "step", 4, 1, ages=3),
        # the large expert, 16 environments: the largest call
        "step_large_b16": _case("large", "step", 4, 16, ages=3),
        # the synchronous baseline: ten passes over one chunk
        "full_pi_b1": _case("pi", "full", 6, 1, euler=10),
        # one micro-batch of the training objective, samples of ten context ages
        "train_pi_b24": _case("pi", "train", 6, 24, ages=10),
        # the same objective in 32 bits (a validation run), small widths
        "train_small_f32_b4": _case("small", "train", 2, 4, ages=4, dtype="f32"),
        # the observation encoder of one robot, called at every tick beside the step
        "encode_pi_b1": _case("pi", "encode", 2, 1),
        # ragged sizes and the optional forms together: relative actions, the offset adapter, rotary positions
        "state_ragged_b5": _case("small", "state", 4, 5, nkv=4, mlp=1360, horizon=21, action_dim=9, prefix=77, fop=5,
                                 ages=3, offset="adapter", rope=10000.0),
    }
    return [dict(c, name=n) for n, c in cases.items()]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """Any family, entry point, depth and batch, slots and prefix from short to the family's own, ragged more often
    than not; never more work than the largest listed case (32-bit models: than a few rows of the small expert)."""
    while True:
        family = rng.choice(["tiny", "small", "pi", "pi", "large"])
        call = rng.choice(["step", "step", "step", "state", "full", "train", "train", "encode"])
        f = FAMILIES[family]
        c = _case(family, call, rng.randint(1, 6), _log_int(rng, 1, 64))
        c["dtype"] = "f32" if family == "tiny" or (family == "small" and rng.random() < 0.3) else "bf16"
        c["horizon"] = _log_int(rng, 4, min(128, 2 * f["horizon"]))
        c["action_dim"] = rng.randint(3, 32)
        c["prefix"] = rng.choice([f["prefix"], rng.randint(0, f["prefix"])])
        c["fop"] = rng.choice([0, f["fop"], rng.randint(1, f["fop"])])
        c["mlp"] = rng.choice([f["mlp"], 16 * rng.randint(f["mlp"] // 32, f["mlp"] // 16)])
        c["offset"] = rng.choice(["mlp", "mlp", "mlp", "concat", "adapter"])
        c["rope"] = rng.choice([0.0, 0.0, 0.0, 10000.0])
        c["ages"] = rng.randint(1, 10)
        if call == "encode":
            c["fop"] = max(c["fop"], 1)
            c["obs"] = 8 * rng.randint(f["obs"] // 16, f["obs"] // 8)
        if call == "full":
            c["euler"] = rng.randint(1, 10)
        if call == "step" and c["batch"] > 4 and rng.random() < 0.5:
            c["refresh"] = rng.randint(3, 6)
        wk = work(c)
        if wk["flops"] < (1.5e9 if c["dtype"] == "f32" else 8e11) and wk["bytes"] < 2e9:
            return c


def _adapters(c):
    return [l for l in range(c["layers"]) if l % 2 == 1 and c["fop"] > 0]


def _weight_shapes(c):
    w, D, hd = c["width"], c["action_dim"], c["hd"]
    qd, kvd = c["nq"] * hd, c["nkv"] * hd
    s = {"in.w": (w, D + (c["offset"] == "concat")), "in.b": (w,), "time.w1": (w, w), "time.b1": (w,),
         "time.w2": (w, w), "time.b2": (w,)}
    if c["offset"] == "mlp":
        s.update({"delta.w1": (w, 1), "delta.b1": (w,), "delta.w2": (w, w), "delta.b2": (w,)})
    if c["offset"] == "adapter":
        s.update({"at.w1": (w, 2 * w + 1), "at.b1": (w,), "at.w2": (w, w), "at.b2": (w,), "ta.w1": (w // 4, 2 * w),
                  "ta.b1": (w // 4,), "ta.w2": (w, w // 4), "ta.alpha": (1,)})
    for l in range(c["layers"]):
        p = "layers.%d." % l
        s.update({p + "mod.w": (6 * w, w), p + "mod.b": (6 * w,), p + "qkv.w": (qd + 2 * kvd, w), p + "o.w": (w, qd),
                  p + "gate.w": (c["mlp"], w), p + "up.w": (c["mlp"], w), p + "down.w": (w, c["mlp"])})
        if l in _adapters(c):
            s.update({p + "fop.gamma": (w,), p + "fop.q.w": (qd, w), p + "fop.kv.w": (2 * kvd, w),
                      p + "fop.o.w": (w, qd), p + "fop.alpha": (1,)})
    s.update({"final.mod.w": (3 * w, w), "final.mod.b": (3 * w,), "out.w": (D, w), "out.b": (D,)})
    if c["fop"] > 0:
        s.update({"fop.w1": (w, c["obs"]), "fop.b1": (w,), "fop.w2": (c["fop"] * w, w), "fop.b2": (c["fop"] * w,)})
    return s


def _round(c, x):
    return x.to(torch.bfloat16).float() if c["dtype"] == "bf16" else x


def _inputs(c, seed):
    """Everything a call reads, on the GPU: weights (32-bit tensors holding the model's precision) and inputs."""
    g = torch.Generator(device=DEV).manual_seed(seed * 2654435761 % (1 << 31) + 1)

    def normal(*shape):
        return torch.randn(shape, generator=g, device=DEV)

    w = c["width"]
    weights = {}
    for name, shp in _weight_shapes(c).items():
        a = normal(*shp) * (1.0 / math.sqrt(shp[1]) if len(shp) == 2 else 0.02)
        if name.endswith("alpha"):
            a.fill_(1.0)
        if name.endswith(".mod.b") and not name.startswith("final"):
            a[2 * w:3 * w] += 1.0
            a[5 * w:6 * w] += 1.0
        weights[name] = _round(c, a)
    B, H, D, L = c["batch"], c["horizon"], c["action_dim"], c["layers"]
    T = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    x = dict(weights=weights, seed=seed)
    if c["call"] == "encode":
        x["obs"] = normal(B, c["obs"])
        return x
    ctx = (B, L, c["prefix"], c["nkv"], c["hd"])
    x["k"], x["v"] = normal(*ctx).to(T), normal(*ctx).to(T)
    x["tokens"] = normal(B, c["fop"], w).to(T) if c["fop"] > 0 else None
    # context ages: refreshed in turn, or a spread of `ages` values
    x["age"] = [c["refresh"] + e % c["refresh"] if c["refresh"] else 1 + e % c["ages"] for e in range(B)]
    if c["call"] in ("full", "train"):
        x["noise"] = normal(B, H, D)
    if c["call"] == "train":
        x["target"] = normal(B, H, D)
    if c["call"] == "state":
        x["robot"] = normal(B, D)
        x["mask"] = [int(d % 3 != 2) for d in range(D)]
    return x


def _config(c):
    return types.SimpleNamespace(
        layers=c["layers"], width=c["width"], n_q_heads=c["nq"], n_kv_heads=c["nkv"], head_dim=c["hd"],
        mlp_dim=c["mlp"], horizon=c["horizon"], action_dim=c["action_dim"], prefix_len=c["prefix"], n_fop=c["fop"],
        fop_obs_dim=c["obs"], fop_stride=2, dtype=ravel.BF16 if c["dtype"] == "bf16" else ravel.F32,
        model_kind=ravel.TRANSFORMER, delta_bias=0.25, rms_eps=1e-6,
        offset_mode={"mlp": 0, "concat": 1, "adapter": 2}[c["offset"]], rope_base=c["rope"])


def prepare(case, seed):
    c = case
    x = _inputs(c, seed)
    model = ravel.Model(_config(c), {n: a.cpu().numpy() for n, a in x.pop("weights").items()})
    buf = ravel.Buffer(model, c["batch"], seed)
    B, H, D, w = c["batch"], c["horizon"], c["action_dim"], c["width"]
    s = dict(x, case=c, model=model, buf=buf, t=0)
    if c["call"] == "encode":
        s["out"] = torch.empty((B, c["fop"], w), device=DEV,
                               dtype=torch.bfloat16 if c["dtype"] == "bf16" else torch.float32)
        return s
    buf.set_option(ravel.OPT_SYNC_CONTEXT, 1)
    if c["prefix"] == 0:  # no prefix tokens: the contexts are empty, their publication still sets the age
        s["k"] = s["v"] = torch.zeros(8, device=DEV)
    for e in range(B):
        k, v = (s["k"][e], s["v"][e]) if c["prefix"] else (s["k"], s["v"])
        buf.set_context(e, k, v, -s["age"][e])
    if c["refresh"]:
        s["producer"] = torch.cuda.Stream()
    if c["call"] in ("step", "state"):
        s["action"] = torch.empty((B, D), device=DEV)
    if c["call"] == "state":
        buf.set_relative_dims(s["mask"])
    if c["call"] == "full":
        s["chunk"] = torch.empty((B, H, D), device=DEV)
    if c["call"] == "train":
        s["ages_dev"] = torch.tensor(s["age"], dtype=torch.int64, device=DEV)
        s["loss"], s["vel"] = torch.empty(B, device=DEV), torch.empty((B, H, D), device=DEV)
    buf.sync()
    return s


def run(state):
    s, c, buf = state, state["case"], state["buf"]
    if c["call"] == "encode":
        buf.fop_encode(s["obs"], s["out"])
        return s["out"]
    if c["call"] == "full":
        buf.full_denoise(c["euler"], s["tokens"], s["noise"], s["chunk"])
        return s["chunk"]
    if c["call"] == "train":
        buf.train_loss(s["target"], s["noise"], s["ages_dev"], s["tokens"], s["loss"], s["vel"])
        return s["loss"], s["vel"]
    t, per = s["t"], c["refresh"]
    if per:  # the environments whose turn it is get a context one period old, from the encoder's stream
        for e in range(-t % per, c["batch"], per):
            i = (e + t) % c["batch"]
            k, v = (s["k"][i], s["v"][i]) if c["prefix"] else (s["k"], s["v"])
            buf.set_context(e, k, v, t - per, stream=s["producer"])
    if c["call"] == "state":
        buf.step_state(s["tokens"], s["robot"], s["action"])
    else:
        buf.step(s["tokens"], s["action"])
    s["t"] = t + 1
    return s["action"]


def _distinct_ages(c):
    return min(c["batch"], c["refresh"] or c["ages"])


def work(case):
    """One pass: weights, contexts and inputs read once (a chunk's Euler passes each read them), outputs written."""
    c = case
    w, D, H, B, L = c["width"], c["action_dim"], c["horizon"], c["batch"], c["layers"]
    el = 2 if c["dtype"] == "bf16" else 4
    if c["call"] == "encode":
        n = w * c["obs"] + c["fop"] * w * w
        return {"bytes": n * el + 4 * (c["fop"] + 1) * w + B * (c["obs"] * 4 + c["fop"] * w * el),
                "flops": 2.0 * B * n}
    qd, kvd, M = c["nq"] * c["hd"], c["nkv"] * c["hd"], B * H
    ad = len(_adapters(c))
    per_row = L * (w * (qd + 2 * kvd) + qd * w + 3 * w * c["mlp"]) + ad * 2 * qd * w + 2 * w * D
    mod = (6 * L + 2) * w * w
    offset = {"mlp": w * w, "concat": 0, "adapter": (2 * w + 1) * w + w * w + 2 * w * (w // 4) + w * (w // 4)}
    fop_kv = ad * 2 * kvd * w
    passes = c["euler"] if c["call"] == "full" else 1
    groups = 1 if c["call"] == "full" else _distinct_ages(c)
    mod_rows = groups if c["call"] == "full" else groups * H
    flops = 2.0 * (M * per_row + mod_rows * mod + B * c["fop"] * fop_kv)
    flops += 2.0 * offset[c["offset"]] * (M if c["offset"] == "adapter" else groups)
    flops += 4.0 * B * H * qd * (L * (c["prefix"] + H) + ad * c["fop"])
    b = (per_row + mod + offset[c["offset"]] + fop_kv) * el
    b += B * (L * c["prefix"] * 2 * kvd + (c["fop"] * w if ad else 0)) * el + 2 * M * D * 4
    if c["call"] == "train":
        b += 2 * M * D * 4
    return {"bytes": passes * b, "flops": passes * flops}


def tolerance(case):
    """About four times what the paths show against 64 bits: velocities are off by up to 6e-3 in bf16 (1.1e-6 in 32
    bits), and a step moves the released action by a velocity over the horizon."""
    c = case
    if c["call"] == "encode":
        return {"rel": 1e-2 if c["dtype"] == "bf16" else 2e-6}
    if c["call"] in ("step", "state"):
        return {"rel": 2.5e-2 / c["horizon"] if c["dtype"] == "bf16" else max(5e-6 / c["horizon"], 4e-7)}
    return {"rel": 2.5e-2 if c["dtype"] == "bf16" else 5e-6}


# --- the same in 64 bits, plain torch -------------------------------------------------------------------------------


def _ring(seed, B, H, D):
    """Initial ring: Philox4x32-10 words keyed by the seed, counter (group of 4, env, action index), Box-Muller."""
    n4 = (D + 3) // 4
    c = np.zeros((B, H, n4, 4), np.uint64)
    c[..., 0] = np.arange(n4)
    c[..., 1] = np.arange(B)[:, None, None]
    c[..., 2] = np.arange(H)[None, :, None]
    m32, s32 = np.uint64(0xFFFFFFFF), np.uint64(32)
    key = [seed & 0xFFFFFFFF, seed >> 32]
    for r in range(10):
        k0, k1 = (np.uint64((key[i] + r * bump) & 0xFFFFFFFF) for i, bump in ((0, 0x9E3779B9), (1, 0xBB67AE85)))
        p0, p1 = np.uint64(0xD2511F53) * c[..., 0], np.uint64(0xCD9E8D57) * c[..., 2]
        c = np.stack([(p1 >> s32) ^ c[..., 1] ^ k0, p1 & m32, (p0 >> s32) ^ c[..., 3] ^ k1, p0 & m32], -1)
    u = (c >> np.uint64(8)).astype(np.float64)
    z = np.empty(u.shape)
    for i in (0, 2):
        rad, ang = np.sqrt(-2.0 * np.log((u[..., i] + 1.0) / 2**24)), 2.0 * np.pi * u[..., i + 1] / 2**24
        z[..., i], z[..., i + 1] = rad * np.cos(ang), rad * np.sin(ang)
    return torch.from_numpy(z.reshape(B, H, -1)[..., :D].astype(np.float32)).to(DEV).double()


def _sinusoid(tau, w):
    om = 10000.0 ** (-torch.arange(w // 2, dtype=torch.float64, device=DEV) / (w // 2))
    arg = 1000.0 * tau[..., None] * om
    return torch.cat([torch.sin(arg), torch.cos(arg)], -1)


def _gelu(x):
    return 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x**3)))


def _rms(x):
    return x / torch.sqrt((x * x).mean(-1, keepdim=True) + 1e-6)


def _silu(x):
    return x * torch.sigmoid(x)


def _attend(c, q, k, v):
    B, Tq, Tk, hd = q.shape[0], q.shape[1], k.shape[1], c["hd"]
    q = q.view(B, Tq, c["nq"], hd).transpose(1, 2).contiguous()
    rep = c["nq"] // c["nkv"]
    k, v = (x.reshape(B, Tk, c["nkv"], hd).transpose(1, 2).repeat_interleave(rep, 1).contiguous() for x in (k, v))
    p = torch.softmax(torch.matmul(q, k.transpose(2, 3).contiguous()) / math.sqrt(hd), -1)
    return torch.matmul(p, v).transpose(1, 2).reshape(B, Tq, -1)


def _rope(c, x, heads):
    B, T, hd = x.shape[0], x.shape[1], c["hd"]
    th = c["rope"] ** (-2.0 * torch.arange(hd // 2, dtype=torch.float64, device=DEV) / hd)
    ang = (c["prefix"] + torch.arange(T, dtype=torch.float64, device=DEV))[:, None, None] * th
    a, b = x.view(B, T, heads, 2, hd // 2).unbind(3)
    return torch.stack([a * ang.cos() - b * ang.sin(), b * ang.cos() + a * ang.sin()], 3).reshape(B, T, -1)


def _velocity(c, W, a, k, v, delta, tokens, tau):
    """The expert on slots a [B, H, D]; delta [B], tau [H]."""

    def lin(x, name, bias=None):
        y = x @ W[name].t()
        return y if bias is None else y + W[bias]

    B, H = a.shape[:2]
    w, qd, kvd, ad = c["width"], c["nq"] * c["hd"], c["nkv"] * c["hd"], _adapters(c)
    ctau = lin(_silu(lin(_sinusoid(tau, w), "time.w1", "time.b1")), "time.w2", "time.b2").expand(B, H, w)
    d = delta[:, None, None].expand(B, H, 1)
    if c["offset"] == "mlp":
        dd = lin(_silu(lin(delta[:, None], "delta.w1", "delta.b1")), "delta.w2", "delta.b2")
        cond = _silu(ctau + dd[:, None])
    else:
        cond = _silu(ctau)
    h = lin(torch.cat([a, d], -1) if c["offset"] == "concat" else a, "in.w", "in.b")
    if c["offset"] == "adapter":
        z = torch.cat([h, _sinusoid(tau, w).expand(B, H, w), d], -1)
        g = lin(_silu(lin(z, "at.w1", "at.b1")), "at.w2", "at.b2")
        z = torch.cat([g, _sinusoid(delta, w)[:, None].expand(B, H, w)], -1)
        h = g + torch.tanh(W["ta.alpha"]) * lin(_silu(lin(z, "ta.w1", "ta.b1")), "ta.w2")
    for l in range(c["layers"]):
        p = "layers.%d." % l
        s1, b1, g1, s2, b2, g2 = lin(cond, p + "mod.w", p + "mod.b").split(w, -1)
        q, ks, vs = lin(_rms(h) * (1 + s1) + b1, p + "qkv.w").split([qd, kvd, kvd], -1)
        if c["rope"] > 0:
            q, ks = _rope(c, q, c["nq"]), _rope(c, ks, c["nkv"])
        kk = torch.cat([k[:, l].double().reshape(B, -1, kvd), ks], 1)
        vv = torch.cat([v[:, l].double().reshape(B, -1, kvd), vs], 1)
        h = h + g1 * lin(_attend(c, q, kk, vv), p + "o.w")
        if l in ad:
            qa = lin(_rms(h) * (1 + W[p + "fop.gamma"]), p + "fop.q.w")
            ka, va = lin(tokens.double(), p + "fop.kv.w").split(kvd, -1)
            h = h + torch.tanh(W[p + "fop.alpha"]) * lin(_attend(c, qa, ka, va), p + "fop.o.w")
        y = _rms(h) * (1 + s2) + b2
        h = h + g2 * lin(_gelu(lin(y, p + "gate.w")) * lin(y, p + "up.w"), p + "down.w")
    sf, bf, _ = lin(cond, "final.mod.w", "final.mod.b").split(w, -1)
    return lin(_rms(h) * (1 + sf) + bf, "out.w", "out.b")


def exact(case, seed):
    c = case
    x = _inputs(c, seed)
    W = {n: a.double() for n, a in x.pop("weights").items()}
    B, H, D = c["batch"], c["horizon"], c["action_dim"]
    if c["call"] == "encode":
        y = _gelu(_round(c, x["obs"]).double() @ W["fop.w1"].t() + W["fop.b1"])
        return (y @ W["fop.w2"].t() + W["fop.b2"]).view(B, c["fop"], -1)
    k, v, tokens = x["k"], x["v"], x["tokens"]
    age = torch.tensor(x["age"], dtype=torch.float64, device=DEV)
    prof = torch.arange(1, H + 1, dtype=torch.float64, device=DEV) / H
    if c["call"] == "full":
        a, S = x["noise"].double(), c["euler"]
        for i in range(S):
            a = a - _velocity(c, W, a, k, v, torch.full_like(age, 0.25), tokens, torch.full_like(prof, (S - i) / S)) / S
        return a
    if c["call"] == "train":
        n, y = x["noise"].double(), x["target"].double()
        vel = _velocity(c, W, prof[:, None] * n + (1 - prof[:, None]) * y, k, v, age / H, tokens, prof)
        return ((vel - (n - y)) ** 2).sum(-1).mean(-1), vel
    # the first step; contexts refreshed before it: environment e takes context e, one period old
    a = _ring(seed, B, H, D)
    out = a[:, 0] - _velocity(c, W, a, k, v, age / H + 0.25, tokens, prof)[:, 0] / H
    return out + torch.tensor(x["mask"], device=DEV) * x["robot"].double() if c["call"] == "state" else out

