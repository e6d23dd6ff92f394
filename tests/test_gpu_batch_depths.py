"""Batches advance up to four steps per launch, 2-D and 3-D grids in loops of their own,
with segment heights chosen per launch: every grid ends with the bits of its own plan at
one (3-D) or two (2-D) steps per launch."""
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu
GRIDS = [((512, 512), 1), ((37, 521), 3), ((5, 40), 1), ((250, 264), 2), ((300, 1201), 3), ((64, 1544), 1),
         ((30, 20, 50), 1), ((64, 64, 64), 1), ((7, 33, 250), 1)]


@pytest.mark.parametrize("carry,engine", [("f16", "sparse"), ("bf16", "sparse"), ("f16", "dense")])
@pytest.mark.parametrize("pick", [range(9), range(6), range(6, 9), [1], [7], [0, 7]])
@pytest.mark.parametrize("graph", [True, False])
def test_batch_depths(carry, engine, pick, graph):
    dt = torch.float16 if carry == "f16" else torch.bfloat16
    torch.manual_seed(3)
    plans, xs, ys, want = [], [], [], []
    steps = [(4, 9, 3, 7, 6, 1, 5, 2, 8)[i] for i in pick]
    for i, n in zip(pick, steps):
        shape, r = GRIDS[i]
        w = si.integer_coeffs(len(shape), r, -3, 3, 20 + i, "box") / 64.0
        x = torch.rand(shape, device="cuda").to(dt)
        kw = dict(carry=carry, engine=engine, **(dict(band_height=8) if len(shape) == 2 else {}))
        own = sp.Plan(w, shape, time_block=2 if len(shape) == 2 else 1, **kw)
        z = torch.empty_like(x)
        own.apply(x, z, n)
        want.append(z)
        plans.append(sp.Plan(w, shape, use_graph=graph, **kw))
        xs.append(x)
        ys.append(torch.full_like(x, 7.0))
    for _ in range(3):
        sp.apply_batch(plans, xs, ys, steps)
        torch.cuda.synchronize()
        for y, z in zip(ys, want):
            assert torch.equal(y, z)
            y.fill_(-3.0)
    zs = [x.clone() for x in xs]
    sp.apply_batch(plans, zs, zs, steps)  # in place
    torch.cuda.synchronize()
    for y, z in zip(zs, want):
        assert torch.equal(y, z)
