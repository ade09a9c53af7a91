"""Renders of at most 512 tiles and more than 8,192 slots, whose instances are
emitted and sorted by tile in one radix pass, against the two-level binning of
the same call (taken where 2^20 instances or more, and 2.5 a slot, are expected:
an instance_hint asks for it): lists bit-exact to the float32 key recipe on both
ways, images bitwise equal, so that the blocks kept with each list entry agree.

The scenes cover the emission's edges: 512 slots to a block, windows of 4,096
positions, runs of many windows in few blocks (cameras among large splats),
every tile shape, ragged views, and the limits of 512 tiles and 2^20 slots.
"""
import numpy as np
import pytest

import synth
from tests import parity
from tests.test_gpu_binning import R  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HINT = 4.0e6


def _views(sizes, radius):
    return [synth.look_at_camera((radius * np.sin(0.9 * k), 0.1, -radius * np.cos(0.9 * k)),
                                 width=w, height=h) for k, (w, h) in enumerate(sizes)]


def _both_ways(R, sc, cams, tile, **kw):
    from paper_2603_02887_amd import nxs
    g = nxs.scene_to_device(sc)
    outs = []
    for hint in (0.0, HINT):
        # (the context's own expectation: the last count, of this same scene)
        outs.append(R.render(g, cams, model=0, tile=tile, instance_hint=hint, **kw))
        torch.cuda.synchronize()
        parity.compare_keys(R, sc, cams, tile_w=tile[0], tile_h=tile[1])
    for a, b in zip(*outs):
        for k in ("rgb", "trans", "overdraw"):
            assert torch.equal(a[k], b[k]), k
    return outs[0]


@pytest.mark.parametrize("order", ["depth_first", "tile_first"])
@pytest.mark.parametrize("tile", [(8, 8), (16, 16), (32, 8)])
@pytest.mark.parametrize("n,radius,log_scale", [
    (8193, 3.0, -4.5), (9000, 0.4, -2.0), (10_240, 1.0, -3.0), (65_537, 0.6, -3.5)])
def test_both_ways(R, n, radius, log_scale, tile, order):  # noqa: F811
    sc = synth.random_scene(n, n, log_scale=(log_scale, 0.4))
    print("case:", n, radius, tile, order, flush=True)
    _both_ways(R, sc, _views([(170, 93), (61, 50)], radius), tile, sort_order=order)


@pytest.mark.parametrize("w,h", [(512, 256), (512, 257), (1, 1), (3, 700)])
def test_sizes_around_512_tiles(R, w, h):  # noqa: F811
    sc = synth.random_scene(5, 12_000, log_scale=(-3.5, 0.5))
    print("case:", w, h, flush=True)
    _both_ways(R, sc, _views([(w, h)], 2.0), (16, 16))


@pytest.mark.parametrize("n", [8193, 65_535, 65_536, 200_001, 800_003, 1_048_576, 1_048_577])
def test_chunk_and_segment_sizes_of_the_binning(R, n):  # noqa: F811
    sc = synth.random_scene(n, n, log_scale=(-4.5, 0.5))
    print("case:", n, flush=True)
    _both_ways(R, sc, _views([(203, 149)], 3.0), (16, 16))


def test_deferred_and_images(R):  # noqa: F811
    """Deferred with too small an expectation, and against the FP64 oracle."""
    from paper_2603_02887_amd import nxs
    sc = synth.random_scene(8, 9_500, log_scale=(-3.0, 0.5))
    cams = _views([(150, 110)], 1.5)
    want = _both_ways(R, sc, cams, (16, 16))
    out = R.render(nxs.scene_to_device(sc), cams, model=0, deferred=True, instance_hint=100.0)
    R.status()
    assert torch.equal(out[0]["rgb"], want[0]["rgb"])
    parity.compare_keys(R, sc, cams)
    parity.compare_view(out[0], sc, cams[0], 0, pixels=parity.sample_pixels(cams[0], 300))
