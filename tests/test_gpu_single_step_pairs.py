"""Single-step launches of paired bands at odd radii run two lines per instruction (plans of
16-bit carries and of fp32 carries without the input split keep operands of both forms)."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si
from gpu_helpers import from_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("carry,split", [("f16", 2), ("bf16", 1), ("f32", 2), ("f32", 3)])
@pytest.mark.parametrize("r", [1, 3])
def test_counts_and_results(oracle_mod, r, carry, split):
    shape, h = (24, 250), 6
    w = si.integer_coeffs(2, r, -2, 2, 3 + r)
    x = si.grid_integer(shape, -2, 2, 9)
    xd = torch.from_numpy(x).to(sp.torch_dtype(carry)).to("cuda:0")
    plan = sp.Plan(w, shape, carry=carry, engine="sparse", split=split, time_block=1, tile_h=h)
    # four segments of three line pairs and r before them, in bodies of four; r + 1
    # instructions per pair and half, twice with the input split, whose launches
    # (four lines per instruction) also stream a pair more where a segment starts at row 2 mod 4
    quad = split == 3
    pairs = [h // 2 + r + (1 if quad and s * h % 4 else 0) for s in range(4)]
    want = sum((n + 3) // 4 * 4 for n in pairs) * 2 * (r + 1) * (2 if quad else 1)
    assert plan.work(1) == (1, want)
    y = torch.empty_like(xd)
    plan.apply(xd, y, 1)
    assert np.array_equal(from_dev(y), oracle_mod.apply(w, x, 1))  # sums of integers up to 196: exact
    # launches of several steps beside single ones in one loop, from the other operands
    both = sp.Plan(w / 64.0, shape, carry=carry, engine="sparse", split=split, time_block=2)
    two = sp.Plan(w / 64.0, shape, carry=carry, engine="sparse", split=split, time_block=2)
    one = sp.Plan(w / 64.0, shape, carry=carry, engine="sparse", split=split, time_block=1)
    a, b, t = (torch.empty_like(xd) for _ in range(3))
    both.apply(xd, a, 3)
    two.apply(xd, t, 2)
    one.apply(t, b, 1)
    assert torch.equal(a, b)
