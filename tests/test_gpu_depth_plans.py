"""Changes of the radix depth sort's plan (three passes for up to 27 varying depth
bits, four beyond) in views of more than 8,192 slots, which the sort in LDS does
not take: a waiting render that sorts and bins again, and a deferred one that is
reported and repeated; single views and several (each a part of its own), binned
in two levels and with the instances emitted.  Bit-exact, as the key recipe has
it."""
import pytest

import synth
from tests import parity
from tests.test_gpu_boundary import _depth_range_scene

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

N = 9001
WAYS = {
    "emitted": ([(96, 80)], (16, 16)),
    "emitted, three views": ([(96, 80), (50, 70), (64, 33)], (16, 16)),
    "cells": ([(640, 480)], (8, 8)),
    "cells, three views": ([(320, 240), (111, 90), (200, 301)], (8, 8)),
}


@pytest.fixture(scope="module")
def nxs():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2603_02887_amd import nxs as m
    return m


def _cameras(sizes):
    return [synth.look_at_camera((0.0, 0.0, -3.0), width=w, height=h) for w, h in sizes]


@pytest.mark.parametrize("way", WAYS)
def test_waiting_renders_sort_and_bin_again(nxs, way):
    sizes, tile = WAYS[way]
    cams = _cameras(sizes)
    narrow, wide = _depth_range_scene(2.1, 15.0, n=N), _depth_range_scene(0.4, 60.0, n=N)
    r = nxs.Renderer(0)
    try:
        for k, sc in enumerate((narrow, narrow, wide, wide, narrow, wide)):
            print("case:", way, k, flush=True)
            g = nxs.scene_to_device(sc)
            out = r.render(g, cams, model=1, tile=tile)
            parity.compare_keys(r, sc, cams, tile_w=tile[0], tile_h=tile[1])
            fresh = nxs.Renderer(0)
            want = fresh.render(g, cams, model=1, tile=tile)
            for a, b in zip(out, want):
                assert torch.equal(a["rgb"], b["rgb"]) and torch.equal(a["trans"], b["trans"])
            fresh.close()
    finally:
        r.close()


@pytest.mark.parametrize("way", WAYS)
def test_deferred_renders_are_reported_and_repeated(nxs, way):
    sizes, tile = WAYS[way]
    cams = _cameras(sizes)
    narrow, wide = _depth_range_scene(2.1, 15.0, n=N), _depth_range_scene(0.4, 60.0, n=N)
    r = nxs.Renderer(0)
    try:
        gn, gw = nxs.scene_to_device(narrow), nxs.scene_to_device(wide)
        want = r.render(gw, cams, model=0, tile=tile)     # capacity for both
        r.render(gn, cams, model=0, tile=tile)            # plans three passes
        out = r.render(gw, cams, model=0, tile=tile, deferred=True)
        with pytest.raises(nxs.NxsError):
            r.status()
        assert all(int(o["overdraw"].sum()) == 0 for o in out)   # nothing composited
        out = r.render(gw, cams, model=0, tile=tile, deferred=True)
        assert r.status() == 0
        for a, b in zip(out, want):
            assert torch.equal(a["rgb"], b["rgb"])
        parity.compare_keys(r, wide, cams, tile_w=tile[0], tile_h=tile[1])
    finally:
        r.close()
