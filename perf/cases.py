"""What the stencil library is timed on: calls as a user's program makes them, through
`Plan.apply` and `apply_batch`, over the sizes, types and options this repository's
workloads, size trend and serving mix use.

`listed()` names the cases, `draw(rng)` makes another one of the same ranges,
`prepare` builds the plans and grids a program holds before the call, `run` is one
pass (a whole time loop), `work` the bytes and operations a pass cannot do without,
and `exact` the same result summed tap by tap in fp64.
"""
import functools
import math

import numpy as np
import torch

import paper_2506_22035_amd as sp

DEVICE = "cuda:0"
BYTES = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}


# ------------------------------------------------------------------ stencils

def _mask(ndim, r, kind):
    off = np.abs(np.indices((2 * r + 1,) * ndim) - r)
    return np.ones(off.shape[1:], bool) if kind == "box" else (off > 0).sum(0) <= 1


@functools.lru_cache(maxsize=None)
def stencil(ndim, r, kind, taps):
    """Taps of sum 1 that no repetition amplifies.  "mean": U[0,1) weights; "heat": the
    explicit heat update (diffusion number 0.1); "gauss" and "signed": weights of both
    signs, N(0,1) and U[-1,1], the first seed whose symbol stays within 1."""
    m = _mask(ndim, r, kind)
    w = np.zeros(m.shape)
    if taps == "heat":
        w[m] = 0.1
        w[(r,) * ndim] = 1.0 - 0.1 * (m.sum() - 1)
        return w
    for seed in range(10000):
        g = np.random.default_rng(seed)
        n = int(m.sum())
        v = g.random(n) if taps == "mean" else g.standard_normal(n) if taps == "gauss" else g.uniform(-1.0, 1.0, n)
        if abs(v.sum()) < 1e-6:
            continue
        w[m] = v / v.sum()
        if taps == "mean" or np.abs(np.fft.fftn(w, (256,) * ndim)).max() <= 1.0 + 1e-9:
            return w
    raise RuntimeError("no stable taps")


# ------------------------------------------------------------------ cases

def _shape(case):
    return tuple(case[k] for k in ("nz", "ny", "nx") if k in case)


def _grids(case):
    """The single grids of a case: dicts with shape, stencil, carry, engine, split, steps."""
    if case["op"] == "apply":
        return [dict(case, shape=_shape(case))]
    if case["op"] == "volumes":
        # one box and one heat update advanced together
        base = dict(carry=case["carry"], engine="auto", split=2, r=1, steps=case["steps"])
        return [dict(base, shape=(case["side_a"],) * 2 + (case["nx_a"],), kind="box", taps="mean"),
                dict(base, shape=(case["side_b"],) * 3, kind="star", taps="heat")]
    # a round of the serving mix: stencils uniform over four, sides log-uniform, 1..100 steps
    rng = np.random.default_rng(case["mix"])
    out = []
    for i in range(case["requests"]):
        pick = (i + case["mix"]) % 4
        if pick == 3:
            s = int(round(math.exp(rng.uniform(math.log(64), math.log(case["max_side_3d"]))) / 16.0)) * 16
            shape, r, kind, taps = (s, s, s), 1, "box", "mean"
        else:
            s = int(round(math.exp(rng.uniform(math.log(512), math.log(case["max_side"]))) / 64.0)) * 64
            shape = (s, s)
            r, kind, taps = [(1, "box", "mean"), (3, "star", "signed"), (3, "box", "gauss")][pick]
        out.append(dict(shape=shape, r=r, kind=kind, taps=taps, carry=case["carry"], engine="auto", split=2,
                        steps=int(rng.integers(1, 101))))
    return out


def _plane(name, ny, nx, r, kind, taps, carry, steps, engine="auto", split=2, field="noise"):
    return dict(name=name, op="apply", ny=ny, nx=nx, r=r, kind=kind, taps=taps, carry=carry, steps=steps,
                engine=engine, split=split, field=field)


def listed():
    return [
        # the smallest call: a small fp64 grid, ten steps, where launches and latency count
        _plane("box2d9p_f64_256", 256, 256, 1, "box", "mean", "f64", 10, engine="direct"),
        # the small end of the size trend and of the serving mix
        _plane("box2d49p_f16_512", 512, 512, 3, "box", "gauss", "f16", 50, field="waves"),
        # an ordinary simulation grid of odd extents, in bfloat16
        _plane("star2d13p_bf16_1021x1533", 1021, 1533, 3, "star", "signed", "bf16", 37),
        # a 3 x 3 update on the paper's mid-size plane
        _plane("box2d9p_f16_4096", 4096, 4096, 1, "box", "mean", "f16", 100),
        # the headline: 49 points, 10240 x 10240, 16-bit state
        _plane("box2d49p_f16_10240", 10240, 10240, 3, "box", "gauss", "f16", 50, field="waves"),
        # the same with the state in fp32 (split operands on the matrix engine)
        _plane("box2d49p_f32carry_10240", 10240, 10240, 3, "box", "gauss", "f32", 50, engine="sparse", split=3,
               field="waves"),
        # plain fp32, no matrix engine: what a program that needs fp32 arithmetic calls
        _plane("star2d13p_f32_8192", 8192, 8192, 3, "star", "signed", "f32", 100, engine="direct"),
        # the widest stencil the paper works with (radius 7)
        _plane("box2d7r_f16_10240", 10240, 10240, 7, "box", "gauss", "f16", 50, field="waves"),
        # the paper's line benchmark on a 16-bit state that is rounded once per launch
        dict(name="line3p_f16_10240000", op="apply", nx=10240000, r=1, kind="box", taps="mean", carry="f16",
             steps=100, engine="sparse", split=3, field="noise"),
        # a line of odd length with its state in fp32
        dict(name="line5p_f32carry_2500001", op="apply", nx=2500001, r=2, kind="box", taps="mean", carry="f32",
             steps=60, engine="sparse", split=3, field="noise"),
        # two volumes advanced together
        dict(name="box3d27p_heat3d_f16", op="volumes", side_a=512, nx_a=512, side_b=256, carry="f16", steps=20),
        # a round of the serving mix
        dict(name="serving_mix_f16", op="mix", mix=3, requests=12, max_side=4096, max_side_3d=256, carry="f16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    family = rng.choice(["plane16", "plane16", "plane32", "direct", "wide", "line", "volumes", "mix"])
    if family == "volumes":
        return dict(op="volumes", side_a=_log(rng, 48, 448), nx_a=_log(rng, 48, 640), side_b=_log(rng, 32, 320),
                    carry=rng.choice(["f16", "bf16"]), steps=rng.randint(1, 20))
    if family == "mix":
        return dict(op="mix", mix=rng.randint(4, 10 ** 6), requests=rng.randint(3, 12), max_side=_log(rng, 768, 4096),
                    max_side_3d=_log(rng, 96, 256), carry=rng.choice(["f16", "bf16"]))
    if family == "line":
        carry = rng.choice(["f16", "bf16", "f32"])
        return dict(op="apply", nx=_log(rng, 20000, 10000000), r=rng.randint(1, 3), kind="box", taps="mean",
                    carry=carry, steps=rng.randint(5, 100), engine="sparse",
                    split=3 if carry == "f32" else rng.choice([2, 3]), field="noise")
    ny, nx, r, kind = _log(rng, 200, 8000), _log(rng, 200, 8000), rng.randint(1, 3), rng.choice(["box", "star"])
    if rng.random() < 0.5:
        nx -= nx % 8  # rows of whole 16-byte chunks, as most programs choose them
    taps, engine, split, steps = rng.choice(["mean", "signed"]), "auto", 2, rng.randint(5, 60)
    if family == "plane16":
        carry = rng.choice(["f16", "bf16"])
    elif family == "plane32":
        carry, engine, split = "f32", "sparse", 3
    elif family == "wide":
        carry, r, kind, taps = rng.choice(["f16", "bf16"]), rng.randint(4, 7), "box", "mean"
    else:
        carry, engine = rng.choice(["f32", "f64"]), "direct"
    if carry == "f64":
        steps = max(1, steps // 2)
    return dict(op="apply", ny=ny, nx=nx, r=r, kind=kind, taps=taps, carry=carry, steps=steps, engine=engine,
                split=split, field=rng.choice(["noise", "waves"]))


# ------------------------------------------------------------------ inputs

def _field(shape, kind, carry, gen):
    """U[0,1) values, or (2-D) the mean of eight plane waves with one per cent of noise."""
    f32 = torch.float64 if carry == "f64" else torch.float32
    x = torch.rand(shape, generator=gen, device=DEVICE, dtype=f32)
    if kind == "waves":
        ny, nx = shape
        a = torch.rand(8, generator=gen, device=DEVICE, dtype=f32) * 0.5 + 0.5
        k = torch.randint(1, 17, (2, 8), generator=gen, device=DEVICE).to(f32)
        ph = torch.rand(8, generator=gen, device=DEVICE, dtype=f32) * (2 * math.pi)
        v = torch.outer(torch.arange(ny, device=DEVICE, dtype=f32) / ny, 2 * math.pi * k[0])
        u = torch.outer(2 * math.pi * k[1], torch.arange(nx, device=DEVICE, dtype=f32) / nx) + ph[:, None]
        x = (x * 2 - 1) * 0.01
        x.addmm_(a * torch.cos(v) / 8, torch.sin(u)).addmm_(a * torch.sin(v) / 8, torch.cos(u))
    return x.to(sp.torch_dtype(carry))


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(1000003 * seed + 17)
    return [_field(g["shape"], g.get("field", "noise"), g["carry"], gen) for g in _grids(case)]


def prepare(case, seed):
    grids = _grids(case)
    xs = _inputs(case, seed)
    plans = [sp.Plan(stencil(len(g["shape"]), g["r"], g["kind"], g["taps"]), g["shape"], carry=g["carry"],
                     engine=g["engine"], split=g["split"]) for g in grids]
    return dict(single=case["op"] == "apply", plans=plans, xs=xs, ys=[torch.empty_like(x) for x in xs],
                steps=[g["steps"] for g in grids])


def run(state):
    if state["single"]:
        state["plans"][0].apply(state["xs"][0], state["ys"][0], state["steps"][0])
        return state["ys"][0]
    sp.apply_batch(state["plans"], state["xs"], state["ys"], state["steps"])
    return list(state["ys"])


def work(case):
    nbytes = flops = 0
    for g in _grids(case):
        n = math.prod(g["shape"])
        nbytes += 2 * n * BYTES[g["carry"]]
        flops += 2 * n * g["steps"] * int(_mask(len(g["shape"]), g["r"], g["kind"]).sum())
    return {"bytes": nbytes, "flops": flops}


# ------------------------------------------------------------------ fp64 results

def _iterate(x, w, steps):
    """`steps` steps in fp64, tap by tap, on a grid with a zero frame of the radius."""
    r, nd = w.shape[0] // 2, x.dim()
    inner = tuple(slice(r, r + n) for n in x.shape)
    a = torch.zeros([n + 2 * r for n in x.shape], dtype=torch.float64, device=x.device)
    b = torch.zeros_like(a)
    a[inner] = x.double()
    taps = [(o, float(w[o])) for o in np.ndindex(*w.shape) if w[o] != 0.0]
    for _ in range(steps):
        dst = b[inner].zero_()
        for o, c in taps:
            dst.add_(a[tuple(slice(o[d], o[d] + x.shape[d]) for d in range(nd))], alpha=c)
        a, b = b, a
    return a[inner].clone()


def exact(case, seed):
    out = [_iterate(x, stencil(len(g["shape"]), g["r"], g["kind"], g["taps"]), g["steps"])
           for g, x in zip(_grids(case), _inputs(case, seed))]
    return out[0] if case["op"] == "apply" else out
