"""spider_plan_info of plans that run in LDS sections (1-D lines) or stream lines through
registers (large 2-D grids on the direct engine) describes the launches that are made."""
import pytest

import paper_2506_22035_amd as sp
import stencil_inputs as si

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,r,deepest", [(5000, 1, 64), (400001, 2, 48), (10240000, 1, 64), (10240000, 3, 48)])
def test_lines(n, r, deepest):
    p = sp.Plan(si.coeffs_uniform01(1, r, 3), (n,), carry="f16", engine="sparse")
    info = p.info()
    halo = deepest * r
    lead = (halo - 8 + 15) // 16 * 16 + 8
    width = (256 * info["tile_h2"] - lead - halo) // 16 * 16  # stored points of a section
    assert p.work(deepest) == (1, -(-n // width) * info["tile_h2"] * deepest)
    width = (256 * info["tile_h"] - 8 - r) // 16 * 16
    assert p.work(1) == (1, -(-n // width) * info["tile_h"])


def test_streamed_grids():
    star = si.coeffs_uniform01(2, 3, 3, "star")
    # of the heights that put 1 .. 8 waves of 9 and 18 strips on each of 1024 SIMDs, the model's best
    for side, h in ((2048, 19), (4096, 37)):
        info = sp.Plan(star, (side, side), carry="f32", engine="direct").info()
        assert (info["time_block"], info["tile_h2"]) == (4, h)
    # one step per launch (49 points): the height of that launch
    info = sp.Plan(si.coeffs_uniform01(2, 3, 3), (1300, 1003), carry="f64", engine="direct").info()
    assert (info["time_block"], info["tile_h"], info["tile_h2"]) == (1, 4, 0)
    # asked-for heights and LDS tiles as before
    assert sp.Plan(star, (2048, 2048), carry="f32", engine="direct", tile_h=20).info()["tile_h"] == 20
    assert sp.Plan(star, (512, 512), carry="f32", engine="direct").info()["tile_h2"] == 0
