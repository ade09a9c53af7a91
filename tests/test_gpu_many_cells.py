"""The two-level binning of few slots over many cells, up to the 4,096 of a call
(eight views of 512 cells), where most cells have one short segment or none, and
around the whole rounds in which the cells' starts are read; against the float32
key recipe, bit for bit."""
import pytest

import synth
from tests import parity
from tests.test_gpu_binning import R  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

# (views, width, height): with 8x8 tiles and cells of 4x4 of them
CASES = {"252": (1, 448, 576), "256": (1, 512, 512), "260": (1, 416, 640), "3094": (7, 520, 810),
         "2048": (4, 1024, 512), "4096": (8, 1024, 512)}


@pytest.mark.parametrize("order", ["depth_first", "tile_first"])
@pytest.mark.parametrize("name", CASES)
def test_few_slots_over_many_cells(R, name, order):  # noqa: F811
    from paper_2603_02887_amd import nxs
    views, w, h = CASES[name]
    sc = synth.random_scene(views, 8_500, log_scale=(-4.5, 0.7))
    cams = synth.orbit_cameras(views, 3.0, w, h)
    print("case:", name, order, flush=True)
    R.render(nxs.scene_to_device(sc), cams, model=1, tile=(8, 8), sort_order=order)
    torch.cuda.synchronize()
    assert parity.compare_keys(R, sc, cams, tile_w=8, tile_h=8) > 0
