"""Depth sorts of small views in LDS against the float32 key recipe, bit-exact:
sizes around the limit, several views, culled slots, and depths that crowd the
sort's bins (all equal, few distinct values, two far clusters), which are
sorted through memory.
"""
import numpy as np
import pytest

import synth
from tests import parity

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def R():
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a GPU")
    from paper_2603_02887_amd import nxs
    r = nxs.Renderer(0)
    yield r
    r.close()


def _depths(sc, kind):
    """Means moved along the first camera's axis (z, looking from z = -3)."""
    z = sc.means[:, 2]
    if kind == "equal":
        z[:] = 0.25
    elif kind == "few":
        z[:] = np.round(z * 3.0) / 3.0
    elif kind == "clusters":
        z[::2] = 1e-4 * z[::2]
        z[1::2] = 40.0 + z[1::2]
        sc.scales[1::2] *= 10.0
    elif kind == "behind":
        z[::3] = -4.0 + 0.1 * z[::3]
    return sc


@pytest.mark.parametrize("kind", ["spread", "equal", "few", "clusters", "behind"])
@pytest.mark.parametrize("n", [1, 2, 63, 1025, 8191, 8192, 8193])
def test_small_view(R, n, kind):
    from paper_2603_02887_amd import nxs
    sc = _depths(synth.random_scene(n, n, log_scale=(-4.0, 0.4)), kind)
    cams = [synth.look_at_camera((0.0, 0.0, -3.0), width=90, height=70)]
    print("case:", n, kind, flush=True)
    R.render(nxs.scene_to_device(sc), cams, model=0)
    torch.cuda.synchronize()
    parity.compare_keys(R, sc, cams)


@pytest.mark.parametrize("kind", ["spread", "few", "behind"])
def test_small_views_of_one_call(R, kind):
    from paper_2603_02887_amd import nxs
    sc = _depths(synth.random_scene(9, 3001, log_scale=(-4.0, 0.4)), kind)
    cams = [synth.look_at_camera((0.0, 0.0, -3.0), width=90, height=70)]
    cams += synth.orbit_cameras(10, 2.5, [64 + 3 * v for v in range(10)], [50] * 10)
    g = nxs.scene_to_device(sc)
    print("case:", kind, flush=True)
    R.render(g, cams, model=2)
    R.render(g, cams, model=2, deferred=True)
    R.status()
    torch.cuda.synchronize()
    parity.compare_keys(R, sc, cams)


def test_every_slot_culled(R):
    from paper_2603_02887_amd import nxs
    sc = synth.random_scene(4, 500)
    sc.means[:, 2] -= 10.0
    cams = [synth.look_at_camera((0.0, 0.0, -3.0), target=(0.0, 0.0, 0.0), width=40, height=30)]
    out = R.render(nxs.scene_to_device(sc), cams, model=0, background=(0.1, 0.2, 0.3))
    torch.cuda.synchronize()
    assert R.counts()[0] == 0
    assert torch.allclose(out[0]["rgb"], torch.tensor([0.1, 0.2, 0.3], device="cuda"))
