"""Depth sorts in LDS of views whose depths crowd the sort's bins, which take its
stable passes, with culled slots among them: against the float32 key recipe, bit
for bit, at sizes around the waves' and the work-group's parts."""
import numpy as np
import pytest

import synth
from tests import parity
from tests.test_gpu_depth import R  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.mark.parametrize("n", [130, 191, 511, 513, 1024, 4097, 8191, 8192])
def test_crowded_and_culled(R, n):  # noqa: F811
    """Two depths far apart; a third of the slots behind the camera."""
    from paper_2603_02887_amd import nxs
    sc = synth.random_scene(n, n, log_scale=(-4.0, 0.4))
    z = sc.means[:, 2]
    z[:] = np.where(np.arange(n) % 7 < 5, 0.25, 30.0)
    z[::3] = -9.0
    sc.scales[z > 1.0] *= 10.0
    cams = [synth.look_at_camera((0.0, 0.0, -3.0), width=90, height=70),
            synth.look_at_camera((0.3, 0.0, -3.0), target=(0.3, 0.0, 0.0), width=40, height=50)]
    print("case:", n, flush=True)
    R.render(nxs.scene_to_device(sc), cams, model=0)
    torch.cuda.synchronize()
    assert parity.compare_keys(R, sc, cams) > 0
