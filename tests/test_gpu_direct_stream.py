"""The direct engine's register-streaming kernel (large 2-D grids, automatic depth):
bit for bit the single steps, which the parity tests tie to the oracle."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu

# wide and tall grids, one strip of columns, rows of every length modulo 4, a grid
# just above the tile kernel's range (single steps) and one of eight levels
SHAPES = [(1300, 1003), (4099, 301), (263, 5001), (9, 140002), (300000, 5), (1025, 1024)]


def _apply(plan, x, steps, alias=False):
    y = x.clone() if alias else torch.empty_like(x)
    plan.apply(y if alias else x, y, steps)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("carry", ["f32", "f64"])
@pytest.mark.parametrize("r", [1, 2, 3])
@pytest.mark.parametrize("kind", ["box", "star"])
def test_equals_single_steps(carry, r, kind):
    w = si.coeffs_uniform01(2, r, 5 + r, kind)
    for shape in SHAPES + ([(5800, 5800)] if r == 1 and carry == "f32" else []):
        x = torch.rand(shape, dtype=sp.torch_dtype(carry), device="cuda:0") - 0.25
        auto = sp.Plan(w, shape, carry=carry, engine="direct")
        single = sp.Plan(w, shape, carry=carry, engine="direct", time_block=1)
        T = auto.info()["time_block"]
        assert (T == 1) == (shape == (1025, 1024) or (r == 3 and kind == "box"))
        for steps in (1, 2 * T - 1, 2 * T + 3):
            ref = _apply(single, x, steps)
            got = _apply(auto, x, steps)
            assert torch.equal(got, ref), (shape, steps, (got != ref).nonzero()[:4].tolist())
        assert torch.equal(_apply(auto, x, 2 * T + 3, alias=True), ref)
        n = auto.work(8 * T + 7)[0]  # whole launches, then one per set bit of the remainder
        assert n == (8 * T + 7) // T + bin((8 * T + 7) % T).count("1")


def test_zero_taps_inside_a_box_keep_single_steps(oracle_mod):
    # taps that are skipped when zero: the old kernel, whatever the size
    w = si.integer_coeffs(2, 2, -1, 1, 4)
    w[0, 1] = 0.0
    w[0, 0] = 1.0
    x = si.grid_integer((1200, 1100), -2, 2, 6)
    plan = sp.Plan(w, x.shape, carry="f64", engine="direct")
    assert plan.info()["time_block"] == 1
    got = _apply(plan, torch.from_numpy(x).double().to("cuda:0"), 3).cpu().numpy()
    assert np.array_equal(got, oracle_mod.apply(w, x, 3))
