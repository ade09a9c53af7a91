"""The backward's per-slot sums where the emissions are nearly or exactly equal,
as on one surface, and where one splat covers many tiles.

The adjoint subtracts emissions (E_i - E_k, or E - L_b behind the splat that
stops an exponential pixel), so an error of the size of |g| |E| shows against
a result of the size of |g| |E_i - E_k|.  The reference runs the appendix
recursions in FP64 on the float32 emissions themselves (degree 0: 1/2 + Y_0 c,
two float32 operations), whose differences are exact in float32.

Tolerance: 2e-5 of the sum of a field's absolute terms.  The splats are round,
so the conic's float32 chain (about 20 operations of 6e-8) leaves alpha
relatively 10 ln 2 x 1.2e-6 = 8e-6 off at alpha_min; the 64-pixel sums and the
projections on g add less than 2e-6.
"""
import numpy as np
import pytest

import synth
from oracle import adjoint as A
from oracle import keys as K
from oracle import operators as O
from oracle import project as P
from tests import adjoint_sums, fd
from tests.test_gpu_backward import H_STEP, R, _gpu_grads  # noqa: F401

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

Y0 = np.float32(0.28209479177387814)


def _scene(spread, seed=3, n=120):
    """Round splats over a small view; colours within `spread` of one colour."""
    rng = np.random.default_rng(seed)
    sc = synth.random_scene(seed, n, mean_lo=-0.8, mean_hi=0.8, log_scale=(-1.7, 0.0),
                            logit=(1.0, 0.5))
    base = np.array([0.7, 0.6, 0.8], np.float32)
    sc.sh[:, 0] = (base - np.float32(0.5)) / Y0
    sc.sh[:, 0] += (spread * rng.uniform(-1.0, 1.0, (n, 3))).astype(np.float32)
    cam = synth.look_at_camera((0, 0, -3.0), width=29, height=22)
    return sc, cam


def _emission(sc):
    return np.float32(0.5) + Y0 * sc.sh[:, 0]


def _sums(sc, cam, op, E, g_rgb, bg, alpha_min, t_eps):
    """Slot sums dLoss/d(aleph, u, v, A, B, C) [n, 6] and of their absolute terms."""
    proj, geom = P.project(sc, cam), K.geometry(sc, cam, alpha_min)
    vis = np.nonzero(geom["visible"])[0]
    order = vis[np.lexsort((vis, geom["depth_bits"][vis]))]
    E4 = np.concatenate([E.astype(np.float64), np.zeros((sc.n, 1))], 1)
    Lb = np.concatenate([np.asarray(bg, np.float64), [1.0]])
    out, mag = np.zeros((sc.n, 6)), np.zeros((sc.n, 6))
    for y, x in np.argwhere(np.any(g_rgb != 0, axis=2)):
        al = P.alpha_at(proj, order, x, y)
        ids, a = order[al >= alpha_min], al[al >= alpha_min]
        if ids.size == 0:
            continue
        d, _ = A.adjoint_sequence(list(a), op, E4[ids], Lb,
                                  np.append(g_rgb[y, x].astype(np.float64), 0.0), 0.0, t_eps)
        dx, dy = x + 0.5 - proj["uv"][ids, 0], y + 0.5 - proj["uv"][ids, 1]
        cA, cB, cC = (proj["conic"][ids, k] for k in range(3))
        da = d * a
        terms = [[da / proj["opacity"][ids]], [da * cA * dx, da * cB * dy],
                 [da * cB * dx, da * cC * dy], [-0.5 * da * dx * dx], [-da * dx * dy],
                 [-0.5 * da * dy * dy]]
        for f, parts in enumerate(terms):
            for t in parts:
                np.add.at(out[:, f], ids, t)
                np.add.at(mag[:, f], ids, np.abs(t))
    return out, mag


def _check(R, sc, cam, op, E, g_rgb, bg, alpha_min, t_eps):  # noqa: F811
    want, mag = _sums(sc, cam, op, E, g_rgb, bg, alpha_min, t_eps)
    got = R.slot_grads(sc.n, 1)[0].astype(np.float64)[:, :6]
    assert (mag > 0).sum() > 100
    err = np.abs(got - want) / (2e-5 * mag + 1e-30)
    print("worst of the tolerance", float(err.max()), flush=True)
    assert err.max() <= 1.0, np.argwhere(err > 1.0)[:5]


def test_linear_splats_of_like_colours(R):  # noqa: F811
    """Emissions within 1e-5 of each other; the upstream gradient at saturated
    pixels alone, where E_k is a splat's emission too."""
    from paper_2603_02887_amd import nxs
    sc, cam = _scene(2e-5)
    g = nxs.scene_to_device(sc)
    out = R.render(g, [cam], model=1, keep_state=True)[0]
    on = (out["trans"].cpu().numpy() == 0) & ~adjoint_sums.ambiguous(sc, cam, O.LINEAR)
    assert on.sum() > 100
    g_rgb = np.random.default_rng(1).normal(size=(cam.height, cam.width, 3)).astype(np.float32)
    g_rgb[~on] = 0.0
    R.backward(g, [torch.from_numpy(g_rgb).cuda()])
    _check(R, sc, cam, O.LINEAR, _emission(sc), g_rgb, (0.0, 0.0, 0.0), 1e-3, None)


def test_linear_splats_of_one_colour(R):  # noqa: F811
    """Saturated pixels of one colour: no geometry gradient at all."""
    from paper_2603_02887_amd import nxs
    sc, cam = _scene(0.0)
    g = nxs.scene_to_device(sc)
    out = R.render(g, [cam], model=1, keep_state=True)[0]
    g_rgb = torch.randn(cam.height, cam.width, 3, device="cuda")
    g_rgb *= (out["trans"] == 0)[..., None]
    assert int((g_rgb != 0).sum()) > 100
    G = R.backward(g, [g_rgb])
    torch.cuda.synchronize()
    for k in ("means", "scales", "quats", "opacities"):
        assert torch.count_nonzero(G[k]) == 0, k
    assert torch.count_nonzero(G["sh"]) > 0


def test_exponential_splats_that_stop_before_a_like_background(R):  # noqa: F811
    """alpha_min 0.1 and t_eps 0.95: the first splat stops every pixel, with only
    the background, within 1e-5 of its colour, behind it."""
    from paper_2603_02887_amd import nxs
    sc, cam = _scene(2e-5)
    bg = tuple(float(v) for v in np.array([0.7, 0.6, 0.8], np.float32))
    g = nxs.scene_to_device(sc)
    R.render(g, [cam], model=0, keep_state=True, background=bg, alpha_min=0.1, t_eps=0.95)
    amb = adjoint_sums.ambiguous(sc, cam, O.EXPONENTIAL, alpha_min=0.1, t_eps=0.95,
                                 background=bg)
    g_rgb = np.random.default_rng(2).normal(size=(cam.height, cam.width, 3)).astype(np.float32)
    g_rgb[amb] = 0.0
    R.backward(g, [torch.from_numpy(g_rgb).cuda()])
    _check(R, sc, cam, O.EXPONENTIAL, _emission(sc), g_rgb, bg, 0.1, 0.95)


@pytest.mark.parametrize("model,op", [(0, O.EXPONENTIAL), (1, O.LINEAR), (3, O.SUPERLINEAR)])
def test_elongated_splats_over_many_tiles(R, model, op):  # noqa: F811
    """Splats of 1 : 50 over 8 to 20 tiles each: every gradient of five of them, element
    by element, against central differences of the FP64 oracle.
    Tolerance: 2e-3 |g| + 1e-3 of the field's largest: the pixel-frame moments of
    a splat whose variances are 1 : 2500 apart carry 6e-8 of the longer one into
    the shorter, 1.5e-4, a few times over (three moments, two products with the
    conic)."""
    sc = synth.random_scene(11, 10, mean_lo=-0.5, mean_hi=0.5, logit=(0.0, 0.7), sh_degree=1)
    sc.scales[:] = np.array([0.5, 0.1, 0.01], np.float32)
    cams = [synth.look_at_camera((0, 0, -3.0), width=90, height=62)]
    F = fd.FrozenLoss(sc, cams, op, t_eps=0.0 if model == 0 else None, seed=model)
    G = _gpu_grads(R, sc, cams, F, model, **({"t_eps": -1.0} if model == 0 else {}))
    p = fd.params_of(sc)
    for field in fd.FIELDS:
        scale = np.abs(G[field]).max()
        for idx in np.ndindex(p[field].shape):
            if idx[0] >= 5 or (field == "sh" and idx[1] > 1):
                continue
            h = H_STEP * (abs(p[field][idx]) if field == "scales" else 1.0)
            want = F.grad_element(p, field, idx, h)
            assert abs(G[field][idx] - want) <= 2e-3 * abs(want) + 1e-3 * scale + 1e-9, \
                (field, idx, G[field][idx], want)
