"""Heights of automatic 2-D plans: the launch model's, or on the largest grids of the dense
engine and of single steps with 16-point bands one round of resident waves, as for plans of
an explicit depth."""
import pytest

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("side,carry,opts,r", [
    (8192, "f16", dict(engine="dense"), 5), (10240, "bf16", dict(engine="dense"), 7),
    (8192, "f32", dict(engine="sparse", split=3), 6), (10240, "f16", dict(engine="dense"), 3)])
def test_largest_grids_run_one_round(side, carry, opts, r):
    w = si.coeffs_uniform01(2, r, 4)
    auto = sp.Plan(w, (side, side), carry=carry, **opts).info()
    fixed = sp.Plan(w, (side, side), carry=carry, time_block=auto["time_block"], **opts).info()
    assert (auto["tile_h"], auto["tile_h2"]) == (fixed["tile_h"], fixed["tile_h2"])
