"""The projection's backward with the coefficients' rows passed through LDS
(degrees 1 and 3, 16-byte aligned arrays) and without (degrees 0 and 2, or
arrays that are not aligned), on counts around one work-group of 256.

Each is compared with central differences of the FP64 oracle along directions
(2e-3 of sum |g . d| + 1e-7, as for the other gradients), and the shifted
arrays with the aligned ones: float atomics add each splat's sums in whatever
order the waves finish, so they agree to float32 rounding (1e-4 relative, 1e-5
of the largest).
"""
import numpy as np
import pytest

import synth
from oracle import operators as O
from tests import fd
from tests.test_gpu_backward import H_STEP, R  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def _grads(R, g, cams, F):
    R.render(g, cams, model=1, keep_state=True)
    w = [F.weights(v) for v in range(len(cams))]
    out = R.backward(g, [torch.from_numpy(a).cuda() for a, _ in w],
                     [torch.from_numpy(b).cuda() for _, b in w])
    torch.cuda.synchronize()
    return {k: v.double().cpu().numpy() for k, v in out.items()}


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("n", [1, 255, 257])
def test_coefficient_rows(R, n, degree):  # noqa: F811
    from paper_2603_02887_amd import nxs
    sc = synth.random_scene(80 + n, n, mean_lo=-0.6, mean_hi=0.6, log_scale=(-2.2, 0.3),
                            logit=(-1.0, 0.7), sh_degree=degree)
    cams = [synth.look_at_camera((0, 0, -3.0), width=17, height=12),
            synth.look_at_camera((1.2, 0.4, -2.6), width=9, height=11)]
    F = fd.FrozenLoss(sc, cams, O.LINEAR, seed=degree)
    g = nxs.scene_to_device(sc)
    G = _grads(R, g, cams, F)
    P = fd.params_of(sc)
    rng = np.random.default_rng(n + degree)
    for field in ("means", "quats", "sh"):
        d = rng.normal(size=P[field].shape)
        want = F.grad_direction(P, {field: d}, H_STEP)
        got = float(np.sum(G[field] * d))
        assert abs(got - want) <= 2e-3 * float(np.sum(np.abs(G[field] * d))) + 1e-7, field
    flat = torch.empty(g["sh"].numel() + 1, device="cuda")
    shifted = dict(g)
    shifted["sh"] = flat[1:].view_as(g["sh"]).copy_(g["sh"])
    assert shifted["sh"].data_ptr() % 16 == 4
    S = _grads(R, shifted, cams, F)
    for k in G:
        np.testing.assert_allclose(S[k], G[k], rtol=1e-4, atol=1e-5 * np.abs(G[k]).max(), err_msg=k)
