"""The backward's per-splat sums where a flush is not full.

A wave adds four pending splats at a time and whatever is left at its end, so
scenes of one to nine splats on views of a few pixels (blocks cut by the image's
edge) reach every remainder.  Each parameter block's gradient is compared with
central differences of the FP64 oracle (tests/fd.py).  Tolerance: 2e-3 of sum
|g . d| + 1e-7 along a direction d: float32 terms of relative rounding ~1e-6
against differences whose own error is below 1e-7.
"""
import numpy as np
import pytest

import synth
from oracle import operators as O
from tests import fd
from tests.test_gpu_backward import H_STEP, R, _gpu_grads  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("model,op", [(0, O.EXPONENTIAL), (1, O.LINEAR), (3, O.SUPERLINEAR)])
@pytest.mark.parametrize("n", [1, 2, 3, 4, 5, 7, 8, 9])
def test_sums_of_few_splats(R, n, model, op):  # noqa: F811
    sc = synth.random_scene(60 + n, n, mean_lo=-0.4, mean_hi=0.4, log_scale=(-1.6, 0.3),
                            logit=(0.0, 0.7), sh_degree=1)
    cams = [synth.look_at_camera((0, 0, -3.0), width=13, height=9),
            synth.look_at_camera((1.2, 0.4, -2.6), width=3, height=19)]
    F = fd.FrozenLoss(sc, cams, op, t_eps=0.0 if model == 0 else None, seed=n)
    G = _gpu_grads(R, sc, cams, F, model, **({"t_eps": -1.0} if model == 0 else {}))
    P = fd.params_of(sc)
    rng = np.random.default_rng(n)
    for field in fd.FIELDS:
        for _ in range(2):
            d = rng.normal(size=P[field].shape)
            if field == "scales":
                d *= P[field]
            want = F.grad_direction(P, {field: d}, H_STEP)
            got = float(np.sum(G[field] * d))
            tol = 2e-3 * float(np.sum(np.abs(G[field] * d))) + 1e-7
            assert abs(got - want) <= tol, (field, got, want)


@pytest.mark.parametrize("n", [1, 6])
def test_pixels_stopped_from_the_start(R, n):  # noqa: F811
    """t_eps > 1: the forward composites nothing, so every gradient is zero."""
    sc = synth.random_scene(5, n, mean_lo=-0.4, mean_hi=0.4, log_scale=(-1.6, 0.3))
    cams = [synth.look_at_camera((0, 0, -3.0), width=13, height=9)]
    F = fd.FrozenLoss(sc, cams, O.EXPONENTIAL, t_eps=0.0, seed=n)
    G = _gpu_grads(R, sc, cams, F, 0, t_eps=1.5)
    for k, v in G.items():
        assert not v.any(), k
