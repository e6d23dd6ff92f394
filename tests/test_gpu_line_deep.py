"""1-D lines advanced many steps per launch in LDS (automatic time_block): the same
bits as launches of the plan's time_block, which the fused 1-D tests tie to single
steps and to the oracle."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu

MODES = [("f16", "sparse", 2, None), ("bf16", "dense", 1, None), ("f16", "sparse", 3, None),
         ("bf16", "sparse", 3, None), ("f16", "dense", 3, None), ("f32", "sparse", 3, "f16"),
         ("f32", "sparse", 2, "bf16"), ("f32", "dense", 3, "bf16")]
# one point, block and section edges, odd ends; 2-, 4- and 8-block sections (the last two lengths)
LENGTHS = [1, 7, 255, 256, 479, 480, 481, 4099, 40007, 400001, 2000003]


def _line(n, carry, seed):
    x = torch.from_numpy(si.grid_uniform01((n,), seed)).to("cuda:0")
    return x.to(sp.torch_dtype(carry))


def _apply(plan, x, steps, alias=False):
    y = x.clone() if alias else torch.empty_like(x)
    plan.apply(y if alias else x, y, steps)
    torch.cuda.synchronize()
    return y


@pytest.mark.parametrize("carry,engine,split,operand", MODES)
@pytest.mark.parametrize("r", [1, 2, 3])
def test_equals_launches_of_the_plans_time_block(carry, engine, split, operand, r):
    w = si.coeffs_uniform01(1, r, 31 + r)
    for n in LENGTHS:
        x = _line(n, carry, n % 1009)
        auto = sp.Plan(w, (n,), carry=carry, engine=engine, split=split, operand=operand)
        tb = auto.info()["time_block"]
        fixed = sp.Plan(w, (n,), carry=carry, engine=engine, split=split, operand=operand, time_block=tb)
        for steps in (1, 2, 3, 15, 48, 65, 131):
            a, b = _apply(auto, x, steps), _apply(fixed, x, steps)
            assert torch.equal(a, b), (n, steps, int((a != b).sum()), (a != b).nonzero()[:4].flatten().tolist())


@pytest.mark.parametrize("carry,split", [("f16", 2), ("f16", 3), ("f32", 3)])
def test_long_line_in_place_and_unaligned_base(carry, split):
    # time_block 4 (from 2^22 points): rounding steps inside and after the last whole block
    n, w = (1 << 22) + 5, si.coeffs_uniform01(1, 1, 8)
    buf = _line(n + 1, carry, 3)
    auto = sp.Plan(w, (n,), carry=carry, engine="sparse", split=split)
    assert auto.info()["time_block"] == 4
    fixed = sp.Plan(w, (n,), carry=carry, engine="sparse", split=split, time_block=4)
    for x in (buf[:n], buf[1:]):
        for steps in (7, 66, 101):
            ref = _apply(fixed, x, steps)
            assert torch.equal(_apply(auto, x, steps), ref)
            assert torch.equal(_apply(auto, x, steps, alias=True), ref)


def test_work_counts_and_long_loops():
    w = si.coeffs_uniform01(1, 1, 8)
    n = 5000
    auto = sp.Plan(w, (n,), carry="f16", engine="sparse")
    fixed = sp.Plan(w, (n,), carry="f16", engine="sparse", time_block=2, use_graph=False)
    assert auto.work(0) == (0, 0) and auto.work(64)[0] == 1 and auto.work(65)[0] == 2
    # 5000 points, radius 1, 64 steps: 14 sections of 2 blocks (368 of 512 points stored),
    # one instruction per block and step
    assert auto.work(64)[1] == 14 * 2 * 64
    x = _line(n, "f16", 5)
    steps = 64 * 600 + 3  # more than 512 launches: replayed bodies, then the remainder
    ref = _apply(fixed, x, steps)
    for _ in range(2):
        assert torch.equal(_apply(auto, x, steps), ref)
    assert torch.equal(_apply(auto, x, 64 * 600 - 61), _apply(fixed, x, 64 * 600 - 61))
