"""Grids whose width is not a multiple of 8: whole 16-byte accesses on rows that start
anywhere, the last element of odd rows by itself.  Every remainder of the width, at the
edges of the strips of every kernel (stored strips of 232, 240, 248 and 256 columns,
256 computed, 264 staged), on integer data, bit for bit against the oracle; nothing is
written outside the grid."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si
from test_gpu_random_sweep import int_taps

pytestmark = pytest.mark.gpu

WIDTHS = sorted(set(range(1, 20)) | {b + d for b in (224, 232, 240, 248, 256, 464, 480, 512) for d in range(-3, 11)})
PLANS = [dict(carry="f16", time_block=1), dict(carry="f16", time_block=2), dict(carry="bf16", time_block=3),
         dict(carry="f16", time_block=4), dict(carry="f16", engine="dense", time_block=3),
         dict(carry="f32", engine="sparse", split=3, time_block=1), dict(carry="f32", engine="sparse", split=3, time_block=2),
         dict(carry="f32", engine="sparse", split=3, time_block=3)]


def _check(oracle_mod, w, shape, opts, steps, seed):
    lim = 2.0 ** 8 if opts["carry"] == "bf16" else 2.0 ** 11 if opts["carry"] == "f16" else 2.0 ** 24
    x = si.grid_integer(shape, -2, 2, seed)
    ref, n = x.astype(np.float64), 0
    while n < steps:
        nxt = oracle_mod.apply(w, ref, 1)
        if np.abs(nxt).max() >= lim:
            break
        ref, n = nxt, n + 1
    assert n >= 1
    dt = sp.torch_dtype(opts["carry"])
    size = int(np.prod(shape))
    xd = torch.from_numpy(x).to("cuda:0").to(dt)
    room = torch.full((size + 64,), 77.0, dtype=dt, device="cuda:0")
    out = room[32:32 + size].view(shape)  # a grid inside a larger buffer
    plan = sp.Plan(w, shape, use_graph=False, **opts)
    plan.apply(xd, out, n)
    torch.cuda.synchronize()
    plan.close()
    got = out.double().cpu().numpy()
    assert np.array_equal(got, ref), (shape, opts, n, np.argwhere(got != ref)[:5])
    assert bool((room[:32] == 77.0).all()) and bool((room[32 + size:] == 77.0).all()), (shape, opts)


@pytest.mark.parametrize("opts", PLANS, ids=lambda o: "-".join(str(v) for v in o.values()))
@pytest.mark.parametrize("r", [1, 2, 3])
def test_planes_of_every_width(oracle_mod, r, opts):
    rng = np.random.default_rng(40 + r)
    w = int_taps(2, r, rng)
    for nx in WIDTHS:
        _check(oracle_mod, w, (11 + nx % 4, nx), opts, opts["time_block"], nx)


@pytest.mark.parametrize("carry,engine,split", [("f16", "sparse", 2), ("bf16", "dense", 2), ("f32", "sparse", 3)])
def test_wide_stencils_and_volumes_of_every_width(oracle_mod, carry, engine, split):
    rng = np.random.default_rng(77)
    w5, w3 = int_taps(2, 5, rng), int_taps(3, 1, rng)
    for nx in WIDTHS:
        opts = dict(carry=carry, engine=engine, split=split)
        _check(oracle_mod, w5, (9, nx), opts, 1, nx)
        _check(oracle_mod, w3, (5, 6, nx), opts, 2, nx + 1)


def test_batches_of_ragged_grids(oracle_mod):
    rng = np.random.default_rng(5)
    shapes = [(9, 301), (12, 255), (7, 237), (8, 1), (5, 6, 263), (4, 7, 37), (10, 480)]
    ws = [int_taps(len(s), 3 if i == 0 else 1, rng) for i, s in enumerate(shapes)]
    xs = [si.grid_integer(s, -2, 2, 60 + i) for i, s in enumerate(shapes)]
    xd = [torch.from_numpy(x).to("cuda:0").half() for x in xs]
    ys = [torch.empty_like(x) for x in xd]
    sp.apply_batch([sp.Plan(w, s, carry="f16") for w, s in zip(ws, shapes)], xd, ys, [2] * len(shapes))
    torch.cuda.synchronize()
    for w, x, y in zip(ws, xs, ys):
        ref = oracle_mod.apply(w, x, 2)
        assert np.abs(ref).max() < 2048 and np.array_equal(y.double().cpu().numpy(), ref), y.shape
