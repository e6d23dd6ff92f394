"""Infinities and NaN.  A matrix instruction multiplies a chunk's whole window, zero taps
included, so beyond the stencil's own reach a non-finite value spreads over the chunks that a
step reads it with; launches of several steps see it from a shorter way off.  What holds for
every depth and tiling: each point that the stencil itself reaches is non-finite, each point
that single steps leave finite is untouched, and a finite result is that of the same grid
without the non-finite value.  The direct engine multiplies nothing beyond the taps."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


def _run(w, x, steps, **opts):
    y = torch.full_like(x, 3.0)
    sp.Plan(w, tuple(x.shape), **opts).apply(x, y, steps)
    torch.cuda.synchronize()
    return y


def _reached(shape, at, reach):
    """Points within `reach` of `at` along every axis (a box stencil of positive taps)."""
    m = torch.ones(shape, dtype=torch.bool, device="cuda:0")
    for d, (n, a) in enumerate(zip(shape, at)):
        i = torch.arange(n, device="cuda:0")
        m &= ((i - a).abs() <= reach).reshape([-1 if e == d else 1 for e in range(len(shape))])
    return m


def _bracket(w, x, at, value, steps, deep, single):
    clean = _run(w, x, steps, **deep)
    x = x.clone()
    x[at] = value
    got, one = _run(w, x, steps, **deep), _run(w, x, steps, **single)
    r = w.shape[0] // 2
    assert not got[_reached(x.shape, at, r * steps)].isfinite().any()
    fin = got.isfinite()
    assert torch.equal(got[fin], clean[fin])
    assert fin[one.isfinite()].all()
    return got, one


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("carry,opts", [("f16", dict(engine="sparse")), ("bf16", dict(engine="dense")),
                                        ("f16", dict(engine="sparse", split=3)),
                                        ("f32", dict(engine="sparse", split=3))])
@pytest.mark.parametrize("r", [1, 2, 3])
def test_lines(r, carry, opts, value):
    # sections of 2 blocks: 512 points, of which the ends are their neighbours' too; places at the
    # line's ends, next to the ends of stored ranges, inside the halos and chunks
    n, w = 4099, si.coeffs_uniform01(1, r, 7) + 0.01
    x = torch.from_numpy(si.grid_uniform01((n,), 5)).to("cuda:0").to(sp.torch_dtype(carry))
    w = w / w.sum()
    for steps in (1, 5, 24):
        for at in (0, 7, 8, 367, 368, 375, 376, 391, 392, 455, 456, 463, 1500, n - 1):
            _bracket(w, x, (at,), value, steps, dict(carry=carry, **opts), dict(carry=carry, time_block=1, **opts))


@pytest.mark.parametrize("r", [4, 5])
def test_wide_planes(r):
    w = si.coeffs_uniform01(2, r, 7) + 0.001
    w = w / w.sum()
    x = torch.from_numpy(si.grid_uniform01((50, 700), 5)).to("cuda:0").half()
    for steps in (2, 3):
        for at in ((0, 0), (20, 224), (20, 231), (20, 232), (20, 239), (20, 240), (21, 248), (49, 699)):
            _bracket(w, x, at, float("inf"), steps, dict(carry="f16"), dict(carry="f16", time_block=1))


@pytest.mark.parametrize("r,carry", [(1, "f32"), (2, "f32"), (3, "f64")])
@pytest.mark.parametrize("kind", ["box", "star"])
def test_streamed_planes_spread_as_single_steps(r, carry, kind):
    w = si.coeffs_uniform01(2, r, 7, kind)
    x = torch.rand((1200, 1003), device="cuda:0").to(sp.torch_dtype(carry))
    for at in ((0, 0), (600, 239), (601, 240), (1199, 1002)):
        x[at] = float("inf")
    for steps in (4, 9):
        deep = _run(w, x, steps, carry=carry, engine="direct")
        one = _run(w, x, steps, carry=carry, engine="direct", time_block=1)
        assert torch.equal(deep.isfinite(), one.isfinite())
        assert torch.equal(deep.nan_to_num(7.0, 8.0, 9.0), one.nan_to_num(7.0, 8.0, 9.0))
