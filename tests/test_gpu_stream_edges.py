"""The streamed form at the edges of its passes: every subspace class, pixels around a workgroup's and around the count
that makes workgroups take a second group, one to four channels, both storage types and the pixel-pair layout."""
import numpy as np
import pytest

from gpu_common import GUARD, TOL_F, TOL_STEP, TOL_U_ELEM, TOL_Y
from oracle import prost_oracle as O

pytestmark = pytest.mark.gpu


def _stored(a, storage):
    from paper_1302_2073_amd.tracker import bf16_bits, bf16_to_f64
    return np.asarray(a, np.float32).astype(np.float64) if storage == "f32" else bf16_to_f64(bf16_bits(a))


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("width,height,channels,k", [(16, 16, 1, 1), (257, 1, 1, 2), (51, 5, 2, 3), (85, 3, 4, 4),
                                                     (64, 8, 3, 5), (64, 8, 3, 8), (513, 1, 3, 10), (171, 3, 1, 12),
                                                     (32, 16, 3, 15), (33, 31, 3, 16), (640, 513, 1, 16),
                                                     (640, 1025, 1, 2)])
def test_streamed_frame_against_the_oracle(width, height, channels, k, storage):
    """Costs, coefficients, angle, U and labels of one frame at the tolerances of the resident form."""
    import torch
    from paper_1302_2073_amd.tracker import Tracker
    P, m = width * height, width * height * channels
    rng = np.random.default_rng([width, height, channels, k])
    A = rng.standard_normal((m, k))
    U = _stored(A @ np.linalg.inv(np.linalg.cholesky(A.T @ A).T), storage)
    y = rng.uniform(0.2, 1.0, k)
    labels = (rng.random(P) < 0.05).astype(np.uint8)
    x = U @ (y + 0.05 * rng.standard_normal(k)) + 0.01 * rng.standard_normal(m)
    fg = np.tile(rng.random(P) < 0.05, channels)
    x[fg] += rng.uniform(0.1, 1.0, int(fg.sum()))
    x = _stored(x, storage)
    prm = O.Params(width, height, channels, k=k, mu=1e-3)
    st = O.State(U.copy(), y.copy(), labels, labels.copy(), 150)
    new, info = O.track_frame(st, x, prm)
    with Tracker(width, height, channels, k, storage=storage) as t:
        t.set_launch(-1)
        t.set_state(U, y, labels, 150)
        t.track(torch.tensor(x, dtype=torch.float32 if storage == "f32" else torch.bfloat16, device="cuda"))
        s = t.stats()
        U1, y1, labels1, n1 = t.get_state()
    assert n1 == 151 and s["cg_steps"] == len(s["f"]) - 1 == prm.cg_iters
    assert np.allclose(s["f"], info.cg.f, rtol=TOL_F, atol=0)
    assert np.linalg.norm(y1 - new.y) <= TOL_Y * np.linalg.norm(new.y)
    if storage == "f32":   # the device's ||pi(eta)||, and with it the step, takes U^T U = I, which rounding to bfloat16 breaks
        assert np.isclose(s["theta"], info.theta, rtol=TOL_STEP, atol=0)
        assert np.abs(U1 - new.U).max() <= TOL_U_ELEM * np.abs(new.U).max()
        r = np.abs(x - new.U @ new.y).reshape(channels, P).max(0)
        sure = np.abs(r - prm.thr) > GUARD
        assert np.array_equal(labels1[sure], new.labels[sure])
