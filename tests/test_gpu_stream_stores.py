"""What the streamed form stores, in both storage types: U within one unit of the storage type and every label outside
the guard band, at the edges of its passes, for steps that move most entries of U.  And its two curvature schedules,
which are one pass."""
import numpy as np
import pytest

from gpu_common import GUARD, TOL_STEP, TOL_U_ELEM
from oracle import prost_oracle as O

pytestmark = pytest.mark.gpu


def _stored(a, storage):
    from paper_1302_2073_amd.tracker import bf16_bits, bf16_to_f64
    return np.asarray(a, np.float32).astype(np.float64) if storage == "f32" else bf16_to_f64(bf16_bits(a))


def _tensor(x, storage):
    import torch
    return torch.tensor(x, dtype=torch.float32 if storage == "f32" else torch.bfloat16, device="cuda")


def _case(width, height, channels, k, storage):
    P, m = width * height, width * height * channels
    rng = np.random.default_rng([width, height, channels, k])
    A = rng.standard_normal((m, k))
    U = _stored(A @ np.linalg.inv(np.linalg.cholesky(A.T @ A).T), storage)
    y = rng.uniform(0.2, 1.0, k)
    labels = (rng.random(P) < 0.05).astype(np.uint8)
    x = U @ (y + 0.05 * rng.standard_normal(k)) + 0.01 * rng.standard_normal(m)
    fg = np.tile(rng.random(P) < 0.05, channels)
    x[fg] += rng.uniform(0.1, 1.0, int(fg.sum()))
    return U, y, labels, _stored(x, storage)


def _geodesic_step(U, x, y, labels, prm):
    """Step 2 at the fitted y with ||pi(eta)||^2 = ||eta||^2 - ||U^T eta||^2, as the device has it: rounding U to
    bfloat16 breaks U^T U = I, on which the oracle's projection rests."""
    eta = O.eta_vector(U, x, y, O.pixel_weights(labels, prm.omega, prm.channels), prm.p, prm.mu, prm.cost)
    a = U.T @ eta
    zeta, nu = np.sqrt(max(eta @ eta - a @ a, 0.0)), np.linalg.norm(y)
    theta = zeta * nu * O.step_size(0, prm.t_init, prm.t_min, prm.i_init)
    coef = (np.cos(theta) - 1.0) * (U @ y) / nu - np.sin(theta) / zeta * (eta - U @ a)
    return theta, U + np.outer(coef, y / nu), x - U @ y - coef * nu


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("width,height,channels,k", [(16, 16, 1, 1), (257, 1, 1, 2), (51, 5, 2, 3), (85, 3, 4, 4),
                                                     (64, 8, 3, 5), (64, 8, 3, 8), (513, 1, 3, 10), (171, 3, 1, 12),
                                                     (32, 16, 3, 15), (33, 31, 3, 16), (640, 513, 1, 16),
                                                     (640, 1025, 1, 2)])
def test_stored_subspace_and_labels(width, height, channels, k, storage):
    from paper_1302_2073_amd.tracker import Tracker
    U, y, labels, x = _case(width, height, channels, k, storage)
    P = width * height
    prm = O.Params(width, height, channels, k=k, mu=1e-3)
    fit, _ = O.track_frame(O.State(U.copy(), y.copy(), labels, labels.copy(), 0), x, prm)
    with Tracker(width, height, channels, k, storage=storage) as t:
        t.set_launch(-1)
        t.set_state(U, y, labels, 0)
        t.track(_tensor(x, storage))
        s = t.stats()
        U1, y1, labels1, _ = t.get_state()
    theta, want, r = _geodesic_step(U, x, fit.y, labels, prm)
    assert np.isclose(s["theta"], theta, rtol=TOL_STEP, atol=0)
    bits = 24 if storage == "f32" else 8
    unit = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), 1e-30))) + 1 - bits)
    assert np.all(np.abs(U1 - want) <= unit + TOL_U_ELEM * np.abs(want).max())
    assert np.mean(U1 != U) > 0.5
    big = np.abs(r).reshape(channels, P).max(0)
    sure = np.abs(big - prm.thr) > GUARD
    assert np.array_equal(labels1[sure], (big >= prm.thr)[sure])


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("width,height,channels,k", [(33, 31, 3, 16), (640, 480, 3, 15)])
def test_curvature_schedules_are_one_pass(width, height, channels, k, storage):
    from paper_1302_2073_amd.tracker import Tracker
    U, y, labels, x = _case(width, height, channels, k, storage)
    out = []
    for schedule in (0, 1):
        with Tracker(width, height, channels, k, storage=storage) as t:
            t.set_launch(-1)
            t.set_curvature(schedule)
            t.set_state(U, y, labels, 150)
            t.track(_tensor(x, storage))
            out.append((t.stats(), t.get_state()))
    assert out[0][0] == out[1][0]
    assert all(np.array_equal(a, b) for a, b in zip(out[0][1], out[1][1]))
