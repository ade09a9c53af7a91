"""The two-level binning against the float32 key recipe, bit-exact, at the edges
of its plans: cells of 4x4, 8x4 and 8x8 tiles, views with too many cells and
calls with too many views (every instance sorted by tile instead), chunks of
every size, slots that cover few and many cells, ragged views, both list
orders; and deferred renders of more instances than expected.
"""
import numpy as np
import pytest

import synth
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SIZES = {
    "one tile": ([(7, 5)], (16, 16), 300),
    "one cell, ragged": ([(61, 50)], (16, 16), 1500),
    "4x4 tiles per cell": ([(333, 251), (64, 64), (150, 97)], (16, 16), 1500),
    "4x4, at 512 cells": ([(1024, 512)], (8, 8), 1500),
    "8x4, past 512 cells": ([(1025, 512)], (8, 8), 1500),
    "8x8": ([(1900, 1000)], (8, 8), 1500),
    "too many cells": ([(2200, 1200)], (8, 8), 1500),
    "64 views": ([(40 + v, 33) for v in range(64)], (16, 16), 257),
    "65 views": ([(40 + v, 33) for v in range(65)], (16, 16), 257),
    "wide tiles": ([(500, 77), (31, 200)], (32, 8), 1025),
}


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2603_02887_amd import nxs
    r = nxs.Renderer(0)
    yield r
    r.close()


def _scene(n, seed=31):
    """Mostly small splats, some that cover whole views."""
    sc = synth.random_scene(seed, n, log_scale=(-3.5, 0.4))
    sc.scales[:: max(1, n // 23)] *= 20.0
    return sc


@pytest.mark.parametrize("order", ["depth_first", "tile_first"])
@pytest.mark.parametrize("name", SIZES)
def test_lists_bit_exact(R, name, order):
    from paper_2603_02887_amd import nxs
    sizes, tile, n = SIZES[name]
    sc = _scene(n)
    cams = synth.orbit_cameras(len(sizes), 3.0, [s[0] for s in sizes], [s[1] for s in sizes])
    g = nxs.scene_to_device(sc)
    print("case:", name, order, flush=True)
    R.render(g, cams, model=1, tile=tile, sort_order=order)
    torch.cuda.synchronize()
    assert parity.compare_keys(R, sc, cams, tile_w=tile[0], tile_h=tile[1]) > 0


@pytest.mark.parametrize("n", [1, 255, 256, 257, 65_535, 65_536, 200_001, 800_003])
def test_chunk_and_segment_sizes(R, n):
    from paper_2603_02887_amd import nxs
    sc = synth.random_scene(n, n, log_scale=(-4.5, 0.5))
    cams = [synth.look_at_camera((0.0, 0.0, -3.0), width=203, height=149)]
    print("case:", n, flush=True)
    R.render(nxs.scene_to_device(sc), cams, model=0)
    torch.cuda.synchronize()
    parity.compare_keys(R, sc, cams)


def test_deferred_beyond_the_expected_count(R):
    """A deferred render of 16 times the instances its launches expect."""
    from paper_2603_02887_amd import nxs
    sc = _scene(5000)
    g = nxs.scene_to_device(sc)
    big = [synth.look_at_camera((0.0, 0.0, -3.0), width=800, height=600)]
    small = [synth.look_at_camera((0.0, 0.0, -9.0), width=96, height=80)]
    print("case: large, small, large deferred", flush=True)
    want = R.render(g, big, model=0)[0]["rgb"].clone()
    R.render(g, small, model=0)
    out = R.render(g, big, model=0, deferred=True, instance_hint=500.0)
    R.status()
    assert torch.equal(out[0]["rgb"], want)
    parity.compare_keys(R, sc, big)
