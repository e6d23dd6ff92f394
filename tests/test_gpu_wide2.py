"""Radius 4 .. 7, 16-bit carry: two steps per launch give the bits of single steps."""
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


SMALL = [(1, 1), (3, 17), (40, 239), (33, 240), (61, 241), (50, 248), (70, 496), (301, 733), (512, 1024)]
LARGE = [(4, 4200001), (65, 262144), (2061, 8193), (4096, 4104)]  # r = 6 from 2^22 points, r = 7 from 2^24


@pytest.mark.parametrize("carry", ["f16", "bf16"])
@pytest.mark.parametrize("r,shape", [(r, s) for r in (4, 5) for s in SMALL] + [(r, s) for r in (6, 7) for s in LARGE])
def test_two_steps(shape, r, carry):
    dt = torch.float16 if carry == "f16" else torch.bfloat16
    w = si.integer_coeffs(2, r, -3, 3, 30 + r, "box") / 128.0
    torch.manual_seed(9)
    x = torch.rand(shape, device="cuda").to(dt)
    x[0, 0] = float("inf") if shape == (61, 241) else 0.5
    for steps in (2, 5):
        want = torch.empty_like(x)
        sp.Plan(w, shape, carry=carry, time_block=1).apply(x, want, steps)
        for h in (0, 1, 7, 32, 64):
            p = sp.Plan(w, shape, carry=carry, tile_h=h)
            assert p.info()["time_block"] == 2
            y = torch.full_like(x, 3.0)
            p.apply(x, y, steps)
            torch.cuda.synchronize()
            assert torch.equal(y.view(torch.int16), want.view(torch.int16)), (h, steps)


@pytest.mark.parametrize("r,shape", [(6, (2048, 2047)), (7, (4096, 4095)), (4, (64, 64))])
def test_one_step_where_it_is_faster(r, shape):
    w = si.integer_coeffs(2, r, -3, 3, 30 + r, "box") / 128.0
    assert sp.Plan(w, shape, carry="f16", time_block=2).info()["time_block"] == 1
    if r > 5:
        assert sp.Plan(w, shape, carry="f16").info()["time_block"] == 1
