"""Paired bands at odd radii: four input lines per matrix instruction.  A launch of any
depth and any segment height (also those whose segments start between two groups of four
lines) gives the bits of single steps rounded in between, and automatic plans give the
bits of the explicit depth they pick."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu
DT = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def run(w, x, steps, **opts):
    y = torch.empty_like(x)
    p = sp.Plan(w, tuple(x.shape), **opts)
    p.apply(x, y, steps)
    torch.cuda.synchronize()
    info = p.info()
    p.close()
    return y, info


def weights(r, kind, seed):
    return si.integer_coeffs(2, r, -3, 3, seed, kind) / 64.0


@pytest.mark.parametrize("carry", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("r", [1, 3])
@pytest.mark.parametrize("shape", [(5, 40), (37, 521), (50, 264)])
def test_depths_and_heights(oracle_mod, shape, r, carry):
    w = weights(r, "box", 7 + r)
    x = torch.from_numpy(si.grid_integer(shape, -8, 8, 3) / 8.0).to(DT[carry]).cuda()
    steps = 12
    kw = dict(carry=carry, engine="sparse", band_height=8)
    base, _ = run(w, x, steps, time_block=2, tile_h=64, **kw)
    # fp64, one operand rounding per value: 2^-11 (2^-8) of the sum of absolute products and
    # one rounding of the result per step; fp32 carry keeps 2^-20 of them
    u = {"f16": 2.0**-10, "bf16": 2.0**-7, "f32": 2.0**-19}[carry]
    ref = x.double().cpu().numpy()
    mag = np.abs(ref)
    for _ in range(steps):
        ref = oracle_mod.apply(w, ref, 1)
        mag = oracle_mod.apply(np.abs(w), mag, 1)
    err = np.abs(base.double().cpu().numpy() - ref)
    assert np.all(err <= 2 * steps * u * mag + 1e-5)
    for T in (1, 2, 3) + ((4,) if carry != "f32" else ()):
        for h in (2, 6, 8, 10, 20):
            y, info = run(w, x, steps, time_block=T, tile_h=h, **kw)
            assert info["time_block"] == T
            if T in (2, 4):
                assert torch.equal(y, base), (T, h)
            else:
                e = np.abs(y.double().cpu().numpy() - ref)
                assert np.all(e <= 2 * steps * u * mag + 1e-5), (T, h)


@pytest.mark.parametrize("carry", ["f16", "f32"])
@pytest.mark.parametrize("r,shape", [(1, (724, 724)), (1, (725, 728)), (1, (2900, 2896)), (2, (2900, 2896)),
                                     (3, (512, 512)), (3, (2048, 2048)), (3, (2900, 2896)), (3, (4099, 4096)),
                                     (2, (5796, 5800)), (5, (700, 480)), (7, (33, 300))])
def test_automatic_plans(r, shape, carry):
    if carry == "f32" and r > 3:
        pytest.skip("one step per launch, as with a 16-bit carry")
    w = weights(r, "star", 11 + r)
    torch.manual_seed(5)
    x = torch.rand(shape, device="cuda").to(DT[carry])
    for steps in (1, 7):
        y, info = run(w, x, steps, carry=carry, engine="sparse")
        z, other = run(w, x, steps, carry=carry, engine="sparse", time_block=info["time_block"], tile_h=64)
        # (explicit depths of wide stencils stay at one step, with the same bits)
        assert other["time_block"] == (info["time_block"] if r <= 3 else 1)
        assert torch.equal(y, z), (info["time_block"], steps)
