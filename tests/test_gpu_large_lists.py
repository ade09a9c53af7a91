"""Instance lists of sizes that only large renders reach.

A view of more than 512 cells emits every instance and sorts them by tile: here
past the sort's switch to 4,096-key chunks (3.5M keys), waiting, and deferred
with an expectation so small that every grid of the tile sort and the ranges
loops beyond it.  Bit-exact against the float32 key recipe.

A call of more than 2^28 slots has no bits to spare in its list entries for the
blocks they cover: 64 and 65 views of 4.2M Gaussians (the second too many for
the binning in two levels), each view compared bitwise with the same view alone,
whose entries have them, and two views' gradients with those of the views alone
(float atomics: 1e-4 relative, 1e-5 of the largest)."""
import numpy as np
import pytest

import synth
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def nxs():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2603_02887_amd import nxs as m
    return m


@pytest.mark.timeout(300)
def test_emitted_instances_past_the_chunk_switch(nxs):
    sc = synth.random_scene(3, 300_000, log_scale=(-4.0, 0.3))
    cams = [synth.look_at_camera((0.0, 0.1, -3.0), width=2200, height=1200)]
    g = nxs.scene_to_device(sc)
    r = nxs.Renderer(0)
    try:
        print("case: waiting", flush=True)
        want = r.render(g, cams, model=1, tile=(8, 8))
        m = parity.compare_keys(r, sc, cams, tile_w=8, tile_h=8)
        assert m > 7 << 19, m
        parity.compare_view(want[0], sc, cams[0], 1, pixels=parity.sample_pixels(cams[0], 200))
        print("case: deferred, 1,000 expected", m, flush=True)
        out = r.render(g, cams, model=1, tile=(8, 8), deferred=True, instance_hint=1000.0)
        assert r.status() == 0
        assert torch.equal(out[0]["rgb"], want[0]["rgb"])
        assert parity.compare_keys(r, sc, cams, tile_w=8, tile_h=8) == m
    finally:
        r.close()


@pytest.mark.timeout(300)
@pytest.mark.parametrize("views", [64, 65])
def test_entries_without_block_bits(nxs, views):
    n = (1 << 28) // 64 + 1
    rng = np.random.default_rng(7)
    sc = synth.random_scene(6, 1 << 15, log_scale=(-3.0, 0.5))
    idx = np.sort(rng.choice(n, sc.n, replace=False))   # the visible ones; culled: opacity 0
    full = {"means": np.zeros((n, 3), np.float32), "scales": np.full((n, 3), 0.01, np.float32),
            "quats": np.tile(np.float32([1, 0, 0, 0]), (n, 1)),
            "opacities": np.zeros(n, np.float32), "sh": np.zeros((n, 1, 3), np.float32)}
    for k, a in full.items():
        a[idx] = getattr(sc, k)
    g = {k: torch.from_numpy(a).cuda() for k, a in full.items()}
    g["sh_degree"] = 0
    cams = synth.orbit_cameras(views, 3.0, [40 + v % 7 for v in range(views)],
                               [30 + v % 5 for v in range(views)])
    assert n * views > 1 << 28
    r, one = nxs.Renderer(0), nxs.Renderer(0)
    pick = (0, views - 1)
    d = [torch.zeros(c.height, c.width, 3, device="cuda") for c in cams]
    for v in pick:
        d[v] = torch.randn(cams[v].height, cams[v].width, 3, device="cuda")
    try:
        print("case:", views, "views", flush=True)
        out = r.render(g, cams, model=3, keep_state=True)
        G = r.backward(g, d)
        torch.cuda.synchronize()
        S = None
        for v in range(0, views) if views == 64 else pick:
            ref = one.render(g, [cams[v]], model=3, keep_state=v in pick)
            for k in ("rgb", "trans", "overdraw"):
                assert torch.equal(out[v][k], ref[0][k]), (v, k)
            if v in pick:
                part = one.backward(g, [d[v]])
                S = part if S is None else {k: S[k] + part[k] for k in S}
        assert float(S["opacities"].abs().max()) > 0
        for k in G:
            scale = float(S[k].abs().max())
            assert torch.allclose(G[k], S[k], rtol=1e-4, atol=1e-5 * scale), k
    finally:
        r.close()
        one.close()
        torch.cuda.empty_cache()
