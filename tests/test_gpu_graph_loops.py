"""Time loops on either side of the number of launches from which they are replayed as a
graph (13 to 512 launches; shorter ones are enqueued launch by launch): captured once per
(in, out, steps) and replayed with eager work in between, every replay equals launches
without graphs."""
import numpy as np
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu

PLANS = [
    ("plane", (130, 261), 3, dict(carry="f16", time_block=2)),
    ("plane f32", (67, 300), 1, dict(carry="f32", engine="sparse", split=3, time_block=3)),
    ("wide", (60, 250), 5, dict(carry="bf16")),
    ("volume", (20, 21, 40), 1, dict(carry="f16")),
    ("line", (5000,), 2, dict(carry="f16", engine="sparse")),
    ("line, one step", (700,), 1, dict(carry="f32", engine="sparse", split=3, time_block=1)),
    ("direct tiles", (90, 70), 1, dict(carry="f64", engine="direct")),
    ("direct single", (30, 41), 4, dict(carry="f32", engine="direct")),
    ("direct streamed", (1200, 1003), 2, dict(carry="f32", engine="direct")),
]


def _steps_of(plan, launches):
    return next(s for s in range(1, 100000) if plan.work(s)[0] == launches)


@pytest.mark.parametrize("name,shape,r,opts", PLANS, ids=[p[0] for p in PLANS])
def test_replays_equal_eager_launches(name, shape, r, opts):
    w = si.coeffs_uniform01(len(shape), r, 12)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(4)
    dt = sp.torch_dtype(opts["carry"])
    x = torch.rand(shape, generator=g, device="cuda:0").to(dt)
    graph = sp.Plan(w, shape, **opts)
    eager = sp.Plan(w, shape, use_graph=False, **opts)
    for launches in (12, 13, 40):
        steps = _steps_of(graph, launches)
        want = torch.empty_like(x)
        eager.apply(x, want, steps)
        out, src = torch.empty_like(x), torch.empty_like(x)
        for k in range(4):  # the first captures, the others replay; new values in the same buffers
            src.copy_(x if k % 2 == 0 else x * 0.5)
            out.fill_(7.0)
            graph.apply(src, out, steps)
            torch.cuda.synchronize()
            ref = want
            if k % 2:
                ref = torch.empty_like(x)
                eager.apply(src, ref, steps)
            _ = (src.float() * 2).sum().item()  # eager work between replays
            assert torch.equal(out, ref), (launches, k)
            assert torch.equal(src, x if k % 2 == 0 else x * 0.5)
        for _ in range(3):  # in place
            out.copy_(x)
            graph.apply(out, out, steps)
            torch.cuda.synchronize()
            assert torch.equal(out, want), launches


def test_more_loops_than_the_cache_holds():
    # 64 graphs per plan: older ones are evicted and captured again
    shape, w = (40, 60), si.coeffs_uniform01(2, 1, 12)
    graph = sp.Plan(w, shape, carry="f16", time_block=1)
    eager = sp.Plan(w, shape, carry="f16", time_block=1, use_graph=False)
    x = torch.rand(shape, device="cuda:0").half()
    out, want = torch.empty_like(x), torch.empty_like(x)
    for steps in list(range(13, 13 + 70)) + [13, 14, 50]:
        assert graph.work(steps)[0] == steps
        graph.apply(x, out, steps)
        eager.apply(x, want, steps)
        torch.cuda.synchronize()
        assert torch.equal(out, want), steps
