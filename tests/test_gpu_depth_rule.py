"""Automatic depth of paired-band plans of radius 2 (even: the bits are those of single steps
at any depth)."""
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,carry,want", [
    ((700, 900), "f16", 2), ((2900, 2896), "f16", 3), ((8192, 8192), "bf16", 3),
    ((8192, 8193), "f16", 4), ((10240, 10240), "bf16", 4), ((10240, 10240), "f32", 3)])
def test_radius_2(shape, carry, want):
    w = si.coeffs_uniform01(2, 2, 4)
    assert sp.Plan(w, shape, carry=carry, engine="sparse").info()["time_block"] == want


def test_radius_2_above_2_to_26_points_equals_single_steps():
    w, shape = si.coeffs_uniform01(2, 2, 4), (8200, 8191)
    x = torch.rand(shape, device="cuda:0").half()
    deep, single = torch.empty_like(x), torch.empty_like(x)
    sp.Plan(w, shape, carry="f16").apply(x, deep, 7)
    sp.Plan(w, shape, carry="f16", time_block=1).apply(x, single, 7)
    assert torch.equal(deep, single)
