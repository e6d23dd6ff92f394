"""Batches around the number of grids from which fewer segment heights are tried: heights never
change results."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("n", [63, 64, 200])
def test_many_grids(n, use_graph):
    rng = np.random.default_rng(n)
    plans, xs, want, steps = [], [], [], []
    for i in range(n):
        ndim = 3 if i % 4 == 3 else 2
        r = 1 if ndim == 3 else 1 + i % 3
        shape = tuple(int(v) for v in rng.integers(1, 40 if ndim == 3 else 330, ndim))
        w = si.integer_coeffs(ndim, r, -2, 2, i) / 64.0
        x = torch.from_numpy(rng.uniform(-1, 1, shape)).half().to("cuda:0")
        k = int(rng.integers(0, 12))
        one = sp.Plan(w, shape, carry="f16", time_block=2 if ndim == 2 else 1)
        y = torch.empty_like(x)
        one.apply(x, y, k)
        plans.append(sp.Plan(w, shape, carry="f16", use_graph=use_graph))
        xs.append(x), want.append(y), steps.append(k)
    outs = [torch.full_like(x, 9.0) for x in xs]
    for _ in range(2):
        sp.apply_batch(plans, xs, outs, steps)
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(outs, want)):
            assert torch.equal(a, b), (i, plans[i].shape, steps[i])
            a.fill_(9.0)
