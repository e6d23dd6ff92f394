"""Automatic plane counts per wave of small volumes give the bits of an explicit height."""
import pytest
import torch

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("opts", [dict(carry="f16"), dict(carry="bf16", engine="dense"),
                                  dict(carry="f32", engine="sparse", split=3)])
@pytest.mark.parametrize("shape", [(1, 1, 1), (64, 64, 64), (7, 33, 250), (100, 101, 301), (255, 256, 256), (256, 256, 256)])
@pytest.mark.parametrize("kind", ["box", "star"])
def test_heights(shape, opts, kind):
    w = si.integer_coeffs(3, 1, -3, 3, 4, kind) / 32.0
    torch.manual_seed(2)
    x = torch.rand(shape, device="cuda").to({"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}[opts["carry"]])
    y, z = torch.empty_like(x), torch.empty_like(x)
    sp.Plan(w, shape, **opts).apply(x, y, 3)
    sp.Plan(w, shape, tile_h=32, **opts).apply(x, z, 3)
    assert torch.equal(y, z)
