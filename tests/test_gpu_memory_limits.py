"""Renders close to the memory they may use: the no-alloc forward's 64 MiB and a
context's workspace limit.  A render that does not fit binned in two levels (few
slots with many instances over large cells) is taken with its instances emitted,
and what the other way of an earlier render left behind makes room."""
import pytest

import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nxs():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2603_02887_amd import nxs as m
    return m


def _limited(nxs, limit):
    r = nxs.Renderer(0, allocator=None)
    assert nxs.lib().nxs_set_workspace_limit(r._ctx, limit) == 0
    return r


def _same(a, b):
    for x, y in zip(a, b):
        for k in ("rgb", "trans", "overdraw"):
            assert torch.equal(x[k], y[k]), k


def _many_instances():
    """6,200 Gaussians of 3.4M instances over 972 cells of 8x8 tiles: 62 MiB where
    every instance is emitted, with a row of 64 tiles for every 64 pairs 73."""
    sc = synth.random_scene(3, 6200, log_scale=(-3.32, 0.3))
    return sc, [synth.look_at_camera((0.2 * k, 0.1, -3.0), width=2246, height=2279)
                for k in range(3)]


def test_noalloc_near_its_scratch(nxs):
    sc, cams = _many_instances()
    g = nxs.scene_to_device(sc)
    r = nxs.Renderer(0)
    try:
        want = r.render(g, cams, model=1)
        assert 3_200_000 < r.counts()[0] < 3_600_000
        outs = [{"rgb": torch.full((c.height, c.width, 3), -1.0, device="cuda"),
                 "trans": torch.full((c.height, c.width), -1.0, device="cuda"),
                 "overdraw": torch.full((c.height, c.width), -1, dtype=torch.int32,
                                        device="cuda")} for c in cams]
        r.render_noalloc(g, cams, outs, model=1)
        torch.cuda.synchronize()
        _same(outs, want)
    finally:
        r.close()


def _least(nxs, g, cams, tile):
    """The least limit (to 4 KiB) under which a context renders the call."""
    lo, hi = 0, 1 << 28
    while hi - lo > 4096:
        mid = (lo + hi) // 2
        r = _limited(nxs, mid)
        try:
            r.render(g, cams, model=1, tile=tile)
            hi = mid
        except nxs.NxsError as e:
            assert e.status == -4
            lo = mid
        finally:
            r.close()
    return hi


@pytest.mark.parametrize("n,views,w,h,tile,most", [
    (100, 1, 1024, 512, (8, 8), 393_216),
    (100, 8, 1024, 512, (8, 8), 3_121_152),
    (300, 64, 100, 80, (8, 8), 4_067_328),
    (2000, 1, 1900, 1000, (8, 8), 14_528_512),
])
def test_least_workspace(nxs, n, views, w, h, tile, most):
    """No more than emitting and sorting every instance needs (`most`, measured on
    these scenes where nothing else was done, to 4 KiB)."""
    sc = synth.random_scene(3, n, log_scale=(-3.5, 0.4))
    cams = synth.orbit_cameras(views, 3.0, w, h)
    least = _least(nxs, nxs.scene_to_device(sc), cams, tile)
    print("least", least, "most", most, flush=True)
    assert least <= most + 4096


def test_one_way_after_the_other_under_a_limit(nxs):
    """A limit that just holds the larger call, taken in turn with one that is
    binned the other way."""
    sc = synth.random_scene(4, 9000, log_scale=(-4.0, 0.4))
    g = nxs.scene_to_device(sc)
    many = [synth.look_at_camera((0.0, 0.0, -3.0), width=1900, height=1000)]
    few = [synth.look_at_camera((0.0, 0.0, -3.0), width=170, height=120)]
    ref = nxs.Renderer(0)
    r = _limited(nxs, max(_least(nxs, g, many, (8, 8)), _least(nxs, g, few, (16, 16))))
    try:
        for _ in range(2):
            for cams, tile in ((many, (8, 8)), (few, (16, 16))):
                want = ref.render(g, cams, model=1, tile=tile)
                _same(r.render(g, cams, model=1, tile=tile), want)
    finally:
        ref.close()
        r.close()
