"""Performance cases of the cached sampler: what a program asks of the library, over the range it is used on.

Whole trajectories (the call a generator makes for each image) and the layers and stages a step consists of,
each through its public entry point. Shapes follow the measured workloads: 16^3 and 32^3 latent grids (4096 and
32768 tokens), width 1024, 16 heads of 64, 1374 condition tokens of width 1024, bf16, and the small float32
model. Late cached steps run a few hundred to a few thousand active tokens; full steps run them all.

All inputs are drawn on the GPU from the case's seed; a model's weights are one fixed draw per architecture,
loaded once and shared by the states that step on it, as a sampling server does.
"""
import functools
import math

import torch

from paper_2511_22533_amd import f3c, synth

DEV = "cuda"
F64 = torch.float64


def listed():
    return [
        # The smallest whole call: an 8^3 float32 model, ten steps with a growing quota. Latency and launches.
        dict(name="trajectory8_f32", kind="steps", grid=8, width=128, depth=2, heads=4, cond=64, cond_width=128,
             dtype="f32", batch=1, steps=10, of=10, eta=1.0, full=3, quota="linear", cached=0.5, guided=False),
        # One image at 16^3 with the 24-block model: condition, modulation plan, 5 full steps, then a logistic
        # quota that ends with 80% of the tokens cached.
        dict(name="trajectory16", kind="steps", grid=16, width=1024, depth=24, heads=16, cond=1374, cond_width=1024,
             dtype="bf16", batch=1, steps=25, of=25, eta=3.0, full=5, quota="logistic", cached=0.8, guided=False),
        # 32^3 with the 12-block model: one full step and four with 70% cached, the 1:4 mix of its 25 steps.
        dict(name="steps32", kind="steps", grid=32, width=1024, depth=12, heads=16, cond=1374, cond_width=1024,
             dtype="bf16", batch=1, steps=5, of=25, eta=3.0, full=1, quota="fixed", cached=0.7, guided=False),
        # Self-attention of a full 32^3 step: the longest sequence there is.
        dict(name="self_attention32", kind="attention", dtype="bf16", heads=16, head_dim=64, batch=1, queries=32768,
             keys=0, ragged=0.0, scaled=True),
        # Self-attention of four samples of a 16^3 batch late in their schedules, each with its own active count.
        dict(name="self_attention16_b4", kind="attention", dtype="bf16", heads=16, head_dim=64, batch=4,
             queries=1639, keys=0, ragged=0.5, scaled=True),
        # Cross-attention of a cached 32^3 step to the image tokens, read from the all-block key/value buffer.
        dict(name="cross_attention32", kind="attention", dtype="bf16", heads=16, head_dim=64, batch=1, queries=9831,
             keys=1374, ragged=0.0, scaled=True),
        # The MLP block (norm + modulation, GELU projection, gated residual projection) of a full 32^3 step ...
        dict(name="mlp32", kind="mlp", dtype="bf16", rows=32768, width=1024),
        # ... and of the last cached steps at 16^3, where one layer is a few microseconds of work.
        dict(name="mlp16_late", kind="mlp", dtype="bf16", rows=820, width=1024),
        # The projections around self-attention (norm + modulation, QKV, gated residual output) of a cached
        # 32^3 step.
        dict(name="projections32", kind="proj", dtype="bf16", rows=9831, width=1024),
        # Scoring and selection of a cached 32^3 step.
        dict(name="select32", kind="select", batch=1, tokens=32768, cached=0.7),
        # What frames the blocks of a cached 32^3 step: gather + embedding, output projection, merge + Euler.
        dict(name="frame32", kind="frame", dtype="bf16", batch=1, grid=32, width=1024, cached=0.7),
        # The dynamic-voxel count that calibrates the schedule: two decoded 64^3 grids packed and compared.
        dict(name="sigma64", kind="sigma", batch=1, grid=64),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["steps", "steps", "attention", "attention", "attention", "mlp", "mlp", "proj", "proj",
                       "select", "frame", "sigma"])
    if kind == "steps":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        width = rng.choice([128, 256] if dtype == "f32" else [256, 512, 1024, 1024])
        guided = rng.random() < 0.3
        full = rng.randint(1, 3)
        return dict(kind=kind, grid=rng.randint(8, 12 if dtype == "f32" else 24), width=width,
                    depth=rng.randint(1, 8), heads=width // rng.choice([32, 64] if dtype == "f32" else [64]),
                    cond=_log(rng, 64, 1374), cond_width=64 * rng.randint(2, 16), dtype=dtype,
                    batch=1 if guided else rng.randint(1, 3), steps=full + rng.randint(1, 5), of=25, eta=3.0,
                    full=full, quota=rng.choice(["fixed", "linear"]), cached=round(rng.uniform(0.3, 0.85), 3),
                    guided=guided)
    if kind == "attention":
        dtype = rng.choice(["bf16"] * 5 + ["f32"])
        batch = rng.randint(1, 4)
        return dict(kind=kind, dtype=dtype, heads=rng.choice([4, 8, 16, 16]),
                    head_dim=rng.choice([32, 64]) if dtype == "f32" else 64, batch=batch,
                    queries=_log(rng, 200, (4096 if dtype == "f32" else 20000) // batch),
                    keys=rng.choice([0, 0, _log(rng, 64, 1374)]), ragged=rng.choice([0.0, 0.3, 0.7]),
                    scaled=rng.random() < 0.7)
    if kind in ("mlp", "proj"):
        dtype = rng.choice(["bf16"] * 6 + ["f32"])
        width = rng.choice([128, 256] if dtype == "f32" else [512, 1024, 1024, 1024, 2048])
        return dict(kind=kind, dtype=dtype, rows=_log(rng, 200, 4096 if dtype == "f32" else 32768), width=width)
    if kind == "select":
        return dict(kind=kind, batch=rng.randint(1, 16), tokens=rng.randint(8, 32) ** 3,
                    cached=round(rng.uniform(0.05, 0.95), 3))
    if kind == "frame":
        return dict(kind=kind, dtype=rng.choice(["bf16", "bf16", "f32"]), batch=rng.randint(1, 4),
                    grid=rng.randint(8, 32), width=rng.choice([256, 512, 1024, 1024]),
                    cached=round(rng.uniform(0.1, 0.9), 3))
    return dict(kind=kind, batch=rng.randint(1, 8), grid=rng.randint(32, 160))


# ------------------------------------------------------------------------------------------------ shared inputs

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(g, *shape, scale=1.0, dtype=torch.float32):
    return (torch.randn(*shape, generator=g, device=DEV) * scale).to(dtype)


def _type(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _code(case):
    return f3c.F3C_BF16 if case["dtype"] == "bf16" else f3c.F3C_F32


def _config(case):
    return synth.ModelConfig(grid=case["grid"], width=case["width"], depth=case.get("depth", 1),
                             heads=case.get("heads", case["width"] // 64), cond_tokens=case.get("cond", 64),
                             cond_width=case.get("cond_width", 64), dtype=case["dtype"])


def _weights(cfg):
    """{name: float32 tensor on the GPU}, N(0, 0.02), of values that the model's type holds exactly."""
    g = _gen(7)
    t = torch.bfloat16 if cfg.dtype == "bf16" else torch.float32
    return {name: _randn(g, *shape, scale=0.02).to(t).float() for name, shape in synth.weight_specs(cfg)}


@functools.lru_cache(maxsize=1)
def _model(cfg):
    return f3c.Model(cfg).load({k: w.cpu().numpy() for k, w in _weights(cfg).items()})


def _quotas(case):
    """Cached tokens of each step that is run."""
    n, full, last = case["grid"] ** 3, case["full"], case["steps"]
    u = lambda k: 1.0 / (1.0 + math.exp(-0.5 * (k - 14.0)))  # noqa: E731
    out = []
    for k in range(1, last + 1):
        if k <= full:
            share = 0.0
        elif case["quota"] == "fixed":
            share = 1.0
        elif case["quota"] == "linear":
            share = (k - full) / (last - full)
        else:
            share = (u(k) - u(full)) / (u(last) - u(full))
        out.append(min(n, int(n * case["cached"] * share)))
    return out


def _lengths(case):
    """Queries of each sample: `queries` on average, the samples spread by +- ragged."""
    b, n, r = case["batch"], case["queries"], case["ragged"]
    return [max(1, int(n * (1 + r * (2 * i / (b - 1) - 1)))) if b > 1 else n for i in range(b)]


def _offsets(lengths):
    out = [0]
    for n in lengths:
        out.append(out[-1] + n)
    return out


# ------------------------------------------------------------------------------------------------------ prepare

def prepare(case, seed):
    g = _gen(seed)
    return {"steps": _prepare_steps, "attention": _prepare_attention, "mlp": _prepare_mlp, "proj": _prepare_proj,
            "select": _prepare_select, "frame": _prepare_frame, "sigma": _prepare_sigma}[case["kind"]](case, g)


def _steps_inputs(case, g):
    cfg, b = _config(case), case["batch"]
    x0 = _randn(g, b, cfg.tokens, 8)
    cond = _randn(g, b, cfg.cond_tokens, cfg.cond_width).to(_type(case)).float()
    return x0, cond


def _prepare_steps(case, g):
    x0, cond = _steps_inputs(case, g)
    state = f3c.State(_model(_config(case)), case["batch"], guided=case["guided"])
    times = [float(t) for t in f3c.time_grid(case["of"], case["eta"])]
    return dict(case=case, state=state, x0=x0, cond=cond, x=torch.empty_like(x0),
                uncond=torch.zeros_like(cond) if case["guided"] else None, times=times, quotas=_quotas(case))


def _attention_inputs(case, g):
    w, t, qs = case["heads"] * case["head_dim"], _type(case), _lengths(case)
    scale = f3c.attention_q_scale(case["head_dim"]) if case["scaled"] else 1.0
    if case["keys"]:      # cross-attention: keys and values of one block of the all-block buffer
        ks = [case["keys"]] * case["batch"]
        q = _randn(g, sum(qs), w, scale=scale, dtype=t)
        kv = _randn(g, sum(ks), 4 * w, dtype=t)
        k, v = kv[:, 2 * w:3 * w], kv[:, 3 * w:]
    else:                 # self-attention: the packed QKV projection
        ks = qs
        qkv = _randn(g, sum(qs), 3 * w)
        qkv[:, :w] *= scale
        qkv = qkv.to(t)
        q, k, v = qkv[:, :w], qkv[:, w:2 * w], qkv[:, 2 * w:]
    return q, k, v, _offsets(qs), _offsets(ks)


def _prepare_attention(case, g):
    q, k, v, qo, ko = _attention_inputs(case, g)
    return dict(case=case, q=q, k=k, v=v, q_off=qo, k_off=ko,
                o=torch.empty(q.shape[0], q.shape[1], dtype=q.dtype, device=DEV),
                work=torch.empty(16 << 20, dtype=torch.uint8, device=DEV))


def _row_inputs(case, g, shapes):
    """Residual rows, shift, scale and gate of the modulation, and (weight, bias) of each projection."""
    d, t = case["width"], _type(case)
    out = dict(h=_randn(g, case["rows"], d), shift=_randn(g, d, scale=0.2), scale=_randn(g, d, scale=0.2),
               gate=_randn(g, d, scale=0.5))
    for name, (n, k) in shapes.items():
        out[name] = _randn(g, n, k, scale=0.02, dtype=t)
        out[name + "_b"] = _randn(g, n, scale=0.02)
    return out


def _mlp_shapes(case):
    d = case["width"]
    return {"fc1": (4 * d, d), "fc2": (d, 4 * d)}


def _proj_shapes(case):
    d = case["width"]
    return {"qkv": (3 * d, d), "o": (d, d)}


def _prepare_mlp(case, g):
    s = _row_inputs(case, g, _mlp_shapes(case))
    r, d, t = case["rows"], case["width"], _type(case)
    return dict(s, case=case, u=torch.empty(r, d, dtype=t, device=DEV),
                hid=torch.empty(r, 4 * d, dtype=t, device=DEV))


def _prepare_proj(case, g):
    s = _row_inputs(case, g, _proj_shapes(case))
    r, d, t = case["rows"], case["width"], _type(case)
    return dict(s, case=case, att=_randn(g, r, d, scale=0.3, dtype=t), u=torch.empty(r, d, dtype=t, device=DEV),
                qkv_out=torch.empty(r, 3 * d, dtype=t, device=DEV))


def _select_inputs(case, g):
    b, n = case["batch"], case["tokens"]
    prev = _randn(g, b, n, 8, scale=0.6)
    # half of the tokens kept their velocity at the step before, as cached tokens do
    fresh = torch.rand(b, n, 1, generator=g, device=DEV) < 0.5
    v = torch.where(fresh, prev + _randn(g, b, n, 8, scale=0.1), prev)
    return v, prev, [int(n * case["cached"])] * b


def _prepare_select(case, g):
    v, prev, c = _select_inputs(case, g)
    b, n = case["batch"], case["tokens"]
    i32 = dict(dtype=torch.int32, device=DEV)
    return dict(case=case, v=v, prev=prev, c=c, idx=torch.empty(sum(n - x for x in c), **i32),
                pos=torch.empty(b, n, **i32), score=torch.empty(b, n, device=DEV),
                work=torch.empty(f3c.select_workspace_bytes(b, n), dtype=torch.uint8, device=DEV))


def _frame_inputs(case, g):
    b, n, d = case["batch"], case["grid"] ** 3, case["width"]
    m = n - int(n * case["cached"])
    idx = torch.stack([torch.randperm(n, generator=g, device=DEV)[:m].sort().values for _ in range(b)])
    pos = torch.full((b, n), -1, dtype=torch.int64, device=DEV)
    pos.scatter_(1, idx, torch.arange(b * m, device=DEV).view(b, m))
    return dict(x=_randn(g, b, n, 8), v_cache=_randn(g, b, n, 8, scale=0.6), rows=_randn(g, b * m, d),
                idx=idx, pos=pos, m=m)


def _prepare_frame(case, g):
    s = _frame_inputs(case, g)
    return dict(s, case=case, model=_model(_config(case)), act_off=[i * s["m"] for i in range(case["batch"] + 1)],
                idx32=s["idx"].reshape(-1).int(), pos32=s["pos"].int(), h=torch.empty_like(s["rows"]),
                v_act=torch.empty(s["rows"].shape[0], 8, device=DEV), v_new=torch.empty_like(s["x"]))


def _prepare_sigma(case, g):
    b, n = case["batch"], case["grid"] ** 3
    nxt = _randn(g, b, n) + torch.linspace(1.5, -1.5, n, device=DEV)
    flip = torch.rand(b, n, generator=g, device=DEV) < 0.01
    prev = torch.where(flip, -nxt, nxt)
    words = (n + 31) // 32
    bits = lambda: torch.empty(b, words, dtype=torch.int32, device=DEV)  # noqa: E731
    return dict(case=case, nxt=nxt, prev=prev, bits_next=bits(), bits_prev=bits(),
                counts=torch.empty(b, dtype=torch.int64, device=DEV))


# ---------------------------------------------------------------------------------------------------------- run

def run(s):
    return _RUN[s["case"]["kind"]](s)


def _run_steps(s):
    case, state, x, times, b = s["case"], s["state"], s["x"], s["times"], s["case"]["batch"]
    x.copy_(s["x0"])
    state.reset()
    state.set_cond(s["cond"])
    if case["guided"]:
        state.set_uncond(s["uncond"])
    state.plan_times(times[:case["steps"]])
    for k, c in enumerate(s["quotas"]):
        t, t_next = times[k], times[k + 1]
        if case["guided"] and t >= 0.5:
            state.guided_step(x, t, t_next, [c] * b if c else None, 3.0)
        elif c:
            state.cached_step(x, t, t_next, [c] * b)
        else:
            state.full_step(x, t, t_next)
    # The velocity caches are not compared: a token that rounding moves across the selection's threshold has
    # another cached velocity altogether, in any two correct implementations.
    return {"x": x}


def _run_attention(s):
    case = s["case"]
    f3c.op_attention(_code(case), case["heads"], case["head_dim"], s["q_off"], s["k_off"], s["q"], s["k"], s["v"],
                     s["o"], workspace=s["work"], q_prescaled=case["scaled"])
    return s["o"]


def _run_mlp(s):
    dt = _code(s["case"])
    f3c.op_ln_mod(dt, s["h"], s["u"], s["shift"], s["scale"])
    f3c.op_gemm(dt, 1, s["u"], s["fc1"], s["fc1_b"], out=s["hid"])
    f3c.op_gemm(dt, 2, s["hid"], s["fc2"], s["fc2_b"], resid=s["h"], gate=s["gate"])
    return {"u": s["u"], "hid": s["hid"], "h": s["h"]}


def _run_proj(s):
    dt = _code(s["case"])
    f3c.op_ln_mod(dt, s["h"], s["u"], s["shift"], s["scale"])
    f3c.op_gemm(dt, 0, s["u"], s["qkv"], s["qkv_b"], out=s["qkv_out"])
    f3c.op_gemm(dt, 2, s["att"], s["o"], s["o_b"], resid=s["h"], gate=s["gate"])
    return {"u": s["u"], "qkv": s["qkv_out"], "h": s["h"]}


def _run_select(s):
    f3c.op_select(s["v"], s["prev"], 0.7, s["c"], s["idx"], s["pos"], score=s["score"], workspace=s["work"])
    return {"idx": s["idx"], "pos": s["pos"], "score": s["score"]}


def _run_frame(s):
    f3c.op_embed(s["model"], s["x"], s["act_off"], s["h"], idx_active=s["idx32"])
    f3c.op_final(s["model"], s["rows"], s["v_act"])
    f3c.op_euler(s["x"], s["v_cache"], s["v_act"], s["pos32"], s["act_off"], 0.7, 0.65, s["v_new"])
    return {"h": s["h"], "v_act": s["v_act"], "x": s["x"], "v_new": s["v_new"]}


def _run_sigma(s):
    f3c.op_pack_occupancy(s["nxt"], s["bits_next"])
    f3c.op_pack_occupancy(s["prev"], s["bits_prev"])
    f3c.op_dynamic_voxels(s["bits_next"], s["bits_prev"], s["counts"])
    return {"next": s["bits_next"], "prev": s["bits_prev"], "counts": s["counts"]}


_RUN = {"steps": _run_steps, "attention": _run_attention, "mlp": _run_mlp, "proj": _run_proj,
        "select": _run_select, "frame": _run_frame, "sigma": _run_sigma}


# --------------------------------------------------------------------------------------------------------- work

def work(case):
    kind = case["kind"]
    es = 2 if case.get("dtype") == "bf16" else 4
    if kind == "steps":
        cfg, b = _config(case), case["batch"]
        d, dc, nc, n = cfg.width, cfg.cond_width, cfg.cond_tokens, cfg.tokens
        passes = 2 if case["guided"] else 1
        flops = passes * 2.0 * b * nc * dc * 2 * d * cfg.depth
        times = _times(case)
        bytes_ = 0.0
        for k, c in enumerate(_quotas(case)):
            p = passes if times[k] >= 0.5 else 1
            m = n - c
            flops += p * b * cfg.depth * (2.0 * m * d * d * 14 + 4.0 * m * m * d + 4.0 * m * nc * d)
            # the latent and both caches, the blocks' weights and the condition's keys and values once a step
            bytes_ += b * n * 8 * 4 * 5 + 14.0 * d * d * cfg.depth * es + p * b * nc * 2.0 * d * cfg.depth * es
        return {"bytes": bytes_, "flops": flops}
    if kind == "attention":
        w, qs = case["heads"] * case["head_dim"], _lengths(case)
        ks = [case["keys"]] * case["batch"] if case["keys"] else qs
        return {"bytes": es * w * 2.0 * (sum(qs) + sum(ks)), "flops": 4.0 * w * sum(q * k for q, k in zip(qs, ks))}
    if kind == "mlp":
        r, d = case["rows"], case["width"]
        return {"bytes": r * d * (4 + 4 + es + 4 * es) + 8.0 * d * d * es, "flops": 16.0 * r * d * d}
    if kind == "proj":
        r, d = case["rows"], case["width"]
        return {"bytes": r * d * (4 + 4 + es + es + 3 * es) + 4.0 * d * d * es, "flops": 8.0 * r * d * d}
    if kind == "select":
        b, n = case["batch"], case["tokens"]
        return {"bytes": b * n * (64 + 4 + 4) + 4.0 * b * (n - int(n * case["cached"])), "flops": 30.0 * b * n}
    if kind == "frame":
        b, n, d = case["batch"], case["grid"] ** 3, case["width"]
        m = b * (n - int(n * case["cached"]))
        return {"bytes": m * (32.0 + 4 + es * d + 4 * d) + m * (4.0 * d + 32) + b * n * (32 * 4 + 4.0),
                "flops": 32.0 * m * d}
    b, n = case["batch"], case["grid"] ** 3
    return {"bytes": 2.0 * b * n * (4 + 1 / 8), "flops": 0}


def tolerance(case):
    kind, low = case["kind"], case.get("dtype") == "bf16"
    if kind in ("select", "sigma"):
        return "exact"             # integer decisions, and float32 scores rounded operation by operation
    if kind == "steps":
        # Rounding also moves a few tokens across the selection's threshold, and their latents are then off by a
        # step's worth of velocity: over the whole bf16 trajectory, 0.019 from 64 bits and 0.020 between two
        # implementations that round elsewhere; 4e-4 over a few steps.
        if not low:
            return {"rel": 4e-6, "max": 1e-3}
        return {"rel": 0.03, "max": 0.99} if case["steps"] == case["of"] else {"rel": 2e-3, "max": 0.3}
    if kind == "attention":    # 3.1e-3 with the probabilities rounded against another reference max
        return {"rel": 1.2e-2, "max": 0.1} if low else {"rel": 4e-6, "max": 1e-4}
    if kind == "frame":
        return {"rel": 2e-6, "max": 1e-4}    # float32 sums of 8 and `width` products
    return {"rel": 3e-3, "max": 0.03} if low else {"rel": 4e-6, "max": 1e-4}


# ---------------------------------------------------------------------------- the same in 64 bits, in plain torch

def _times(case):
    """t_k = eta u / (1 + (eta - 1) u) with u = 1 - (k - 1) / T, k = 1 .. T + 1."""
    us = [1.0 - k / case["of"] for k in range(case["of"] + 1)]
    return [case["eta"] * u / (1.0 + (case["eta"] - 1.0) * u) for u in us]


def _norm(h):
    c = h - h.mean(-1, keepdim=True)
    return c / torch.sqrt((c * c).mean(-1, keepdim=True) + 1e-6)


def _gelu(x):
    return 0.5 * x * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (x + 0.044715 * x ** 3)))


def _attend(q, k, v, heads, scale):
    out = torch.empty_like(q)
    hd = q.shape[1] // heads
    for i in range(heads):
        c = slice(i * hd, (i + 1) * hd)
        kt, vh = k[:, c].t().contiguous(), v[:, c].contiguous()
        for r in range(0, q.shape[0], 8192):
            p = torch.softmax((q[r:r + 8192, c] * scale) @ kt, dim=-1)
            out[r:r + 8192, c] = p @ vh
    return out


def exact(case, seed):
    g = _gen(seed)
    return {"steps": _exact_steps, "attention": _exact_attention, "mlp": _exact_mlp, "proj": _exact_proj,
            "select": _exact_select, "frame": _exact_frame, "sigma": lambda c, g: None}[case["kind"]](case, g)


def _exact_attention(case, g):
    q, k, v, qo, ko = _attention_inputs(case, g)
    scale = math.log(2.0) if case["scaled"] else 1.0 / math.sqrt(case["head_dim"])
    return torch.cat([_attend(q[qo[b]:qo[b + 1]].to(F64), k[ko[b]:ko[b + 1]].to(F64), v[ko[b]:ko[b + 1]].to(F64),
                              case["heads"], scale) for b in range(case["batch"])])


def _exact_mlp(case, g):
    s = {k: v.to(F64) for k, v in _row_inputs(case, g, _mlp_shapes(case)).items()}
    u = _norm(s["h"]) * (1.0 + s["scale"]) + s["shift"]
    hid = _gelu(u @ s["fc1"].t() + s["fc1_b"])
    return {"u": u, "hid": hid, "h": s["h"] + s["gate"] * (hid @ s["fc2"].t() + s["fc2_b"])}


def _exact_proj(case, g):
    s = {k: v.to(F64) for k, v in _row_inputs(case, g, _proj_shapes(case)).items()}
    att = _randn(g, case["rows"], case["width"], scale=0.3, dtype=_type(case)).to(F64)
    u = _norm(s["h"]) * (1.0 + s["scale"]) + s["shift"]
    return {"u": u, "qkv": u @ s["qkv"].t() + s["qkv_b"], "h": s["h"] + s["gate"] * (att @ s["o"].t() + s["o_b"])}


def _score(v, prev, t):
    """Stability score of each token: 0.7 norm(|v - prev|) + 0.3 norm(|v|), operation by operation in type t."""
    def magnitude(a):
        s = torch.zeros_like(a[..., 0])
        for c in range(8):
            s = s + a[..., c] * a[..., c]
        return torch.sqrt(s)

    def unit(a):
        lo, hi = a.amin(-1, keepdim=True), a.amax(-1, keepdim=True)
        return (a - lo) / (hi - lo)

    w = torch.tensor(0.7, dtype=torch.float32).to(t)
    v, prev = v.to(t), prev.to(t)
    return w.item() * unit(magnitude(v - prev)) + (torch.tensor(1.0) - w.float()).to(t).item() * unit(magnitude(v))


def _exact_select(case, g):
    v, prev, _ = _select_inputs(case, g)
    return {"idx": None, "pos": None, "score": _score(v, prev, F64)}


def _exact_frame(case, g):
    s, w = _frame_inputs(case, g), {k: v.to(F64) for k, v in _weights(_config(case)).items()}
    x, idx = s["x"].to(F64), s["idx"]
    h = torch.cat([x[b, i] @ w["in_w"].t() + w["in_b"] + w["pos"][i] for b, i in enumerate(idx)])
    v_act = _norm(s["rows"].to(F64)) @ w["out_w"].t() + w["out_b"]
    v = s["v_cache"].to(F64)
    for b, i in enumerate(idx):
        v[b, i] = v_act[b * s["m"]:(b + 1) * s["m"]]
    return {"h": h, "v_act": v_act, "x": x - (0.7 - 0.65) * v, "v_new": v}


def _exact_steps(case, g):
    cfg, n = _config(case), case["grid"] ** 3
    x, cond = (a.to(F64) for a in _steps_inputs(case, g))
    w = {k: v.to(F64) for k, v in _weights(cfg).items()}
    times, d = _times(case), cfg.width
    lin = lambda a, name: a @ w[name + "_w"].t() + w[name + "_b"]  # noqa: E731

    def keys(c):
        return [lin(c, "blk%d.kv" % l) for l in range(cfg.depth)]

    def velocity(xa, idx, t, kv):
        arg = 1000.0 * t * torch.pow(10000.0, -torch.arange(128, dtype=F64, device=DEV) / 128)
        temb = lin(torch.nn.functional.silu(lin(torch.cat([arg.cos(), arg.sin()]), "t1")), "t2")
        h = lin(xa, "in") + w["pos"][idx]
        for l in range(cfg.depth):
            p = "blk%d." % l
            sh1, sc1, g1, sh2, sc2, g2 = lin(torch.nn.functional.silu(temb), p + "mod").view(6, d)
            qkv = lin(_norm(h) * (1.0 + sc1) + sh1, p + "qkv")
            sa = _attend(qkv[:, :d], qkv[:, d:2 * d], qkv[:, 2 * d:], cfg.heads, 1.0 / math.sqrt(cfg.head_dim))
            h = h + g1 * lin(sa, p + "o")
            ca = _attend(lin(_norm(h), p + "q"), kv[l][:, :d], kv[l][:, d:], cfg.heads, 1.0 / math.sqrt(cfg.head_dim))
            h = h + lin(ca, p + "co")
            h = h + g2 * lin(_gelu(lin(_norm(h) * (1.0 + sc2) + sh2, p + "fc1")), p + "fc2")
        return lin(_norm(h), "out")

    out = []
    for b in range(case["batch"]):
        kv, kv0 = keys(cond[b]), keys(torch.zeros_like(cond[b])) if case["guided"] else None
        xb, v, prev = x[b], torch.zeros_like(x[b]), torch.zeros_like(x[b])
        for k, c in enumerate(_quotas(case)):
            t = times[k]
            idx = torch.arange(n, device=DEV)
            if c:   # the selection is taken in float32; a stable sort breaks ties by the token's index
                order = torch.argsort(_score(v.float().cpu(), prev.float().cpu(), torch.float32), stable=True)
                idx = order[c:].sort().values.to(DEV)
            fresh = velocity(xb[idx], idx, t, kv)
            if case["guided"] and t >= 0.5:
                fresh = 4.0 * fresh - 3.0 * velocity(xb[idx], idx, t, kv0)
            new = v.clone()
            new[idx] = fresh
            v, prev = new, v
            xb = xb - (t - times[k + 1]) * v
        out.append(xb)
    return {"x": torch.stack(out)}
