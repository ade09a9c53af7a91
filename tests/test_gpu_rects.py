"""Rectangles in one word and in two: views at and beyond the widest and the
tallest grid of 8x8 blocks that one word holds (255), in every tile shape and
both list orders, and small views (sorted in LDS) beside radix-sorted ones.
Lists and rectangles are compared bit for bit with the float32 key recipe."""
import pytest

import synth
from tests import parity
from tests.test_gpu_binning import R, _scene  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

VIEWS = {
    "254 x 1": [(2032, 8)],
    "255 x 2": [(2040, 9)],
    "256 x 1": [(2041, 7)],
    "1 x 255": [(5, 2040)],
    "2 x 256": [(16, 2041)],
    "one beyond, one within": [(2100, 40), (64, 48)],
}


@pytest.mark.parametrize("order", ["depth_first", "tile_first"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 8)])
@pytest.mark.parametrize("name", VIEWS)
def test_rectangles_bit_exact(R, name, tile, order):  # noqa: F811
    from paper_2603_02887_amd import nxs
    n = 9001 if tile == (16, 16) else 700
    sc = _scene(n)
    cams = [synth.look_at_camera((0.1 * k, 0.0, -3.0), width=w, height=h,
                                 fov_x_deg=60.0 if w >= h else 2.0)
            for k, (w, h) in enumerate(VIEWS[name])]
    print("case:", name, tile, order, flush=True)
    R.render(nxs.scene_to_device(sc), cams, model=1, tile=tile, sort_order=order)
    torch.cuda.synchronize()
    assert parity.compare_keys(R, sc, cams, tile_w=tile[0], tile_h=tile[1]) > 0
