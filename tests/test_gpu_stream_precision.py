"""Precision of the streamed form's reductions: a CG step along a direction that only foreground pixels carry (the
curvature is what is left of entries millions of times larger), and sums whose terms cancel over the pixel groups of a
workgroup."""
import numpy as np
import pytest

from gpu_common import TOL_F, TOL_STEP, TOL_Y
from oracle import prost_oracle as O

pytestmark = pytest.mark.gpu


def _stored(a, storage):
    from paper_1302_2073_amd.tracker import bf16_bits, bf16_to_f64
    return np.asarray(a, np.float32).astype(np.float64) if storage == "f32" else bf16_to_f64(bf16_bits(a))


def _tensor(x, storage):
    import torch
    return torch.tensor(x, dtype=torch.float32 if storage == "f32" else torch.bfloat16, device="cuda")


def _hadamard(k):
    H = np.ones((1, 1))
    while len(H) < k:
        H = np.block([[H, H], [H, -H]])
    return H / np.sqrt(k)


@pytest.mark.parametrize("schedule", [0, 1])
@pytest.mark.parametrize("width,height,channels,k,storage", [(640, 480, 3, 15, "f32"), (1280, 240, 1, 4, "f32"),
                                                             (640, 480, 3, 16, "f32"), (640, 480, 3, 4, "bf16"),
                                                             (641, 481, 1, 16, "bf16"), (640, 480, 3, 16, "bf16"),
                                                             (640, 480, 3, 2, "f32"), (640, 480, 3, 5, "f32"),
                                                             (640, 480, 3, 8, "f32"), (640, 480, 3, 10, "f32")])
def test_step_along_a_direction_of_foreground_pixels(width, height, channels, k, storage, schedule):
    """The background is fitted exactly (r = 0, weight 1, the largest c), so g comes from the foreground pixels alone
    (weight 5e-5), along a direction that every background row of U is orthogonal to: exactly for the dyadic rotations
    (k = 4, 16), to float32 rounding of U otherwise.  d^T H d is about 1e-7 of H's entries times |d|^2."""
    from paper_1302_2073_amd.tracker import Tracker
    P, m = width * height, width * height * channels
    rng = np.random.default_rng([width, k])
    labels = (rng.random(P) < 0.03).astype(np.uint8)
    fg = np.tile(labels.astype(bool), channels)
    A = np.zeros((m, k))
    A[~fg, :k - 1] = rng.integers(-3, 4, (int((~fg).sum()), k - 1))
    A[fg, k - 1] = rng.choice([-2.0, -1.0, 1.0, 2.0], int(fg.sum()))
    if k in (4, 16):
        U = A @ _hadamard(k)
    else:
        U = A @ np.linalg.qr(rng.standard_normal((k, k)))[0]
    U = _stored(U / 1024.0, storage)
    x = np.zeros(m)
    x[fg] = rng.uniform(0.3, 1.0, int(fg.sum()))
    x = _stored(x, storage)
    prm = O.Params(width, height, channels, k=k, mu=1e-3, cg_iters=1)
    new, info = O.track_frame(O.State(U.copy(), np.zeros(k), labels, labels.copy(), 150), x, prm)
    with Tracker(width, height, channels, k, storage=storage, cg_iters=1, mu=1e-3) as t:
        t.set_launch(-1)
        t.set_curvature(schedule)
        t.set_state(U, np.zeros(k), labels, 150)
        t.track(_tensor(x, storage))
        s = t.stats()
        y = t.get_state()[1]
    assert s["cg_steps"] == 1
    assert np.isclose(s["alpha"][0], info.cg.alpha[0], rtol=TOL_STEP, atol=0)
    assert np.allclose(s["f"], info.cg.f, rtol=TOL_F, atol=0)
    assert np.linalg.norm(y - new.y) <= TOL_Y * np.linalg.norm(new.y)


@pytest.mark.parametrize("k", [1, 5, 8, 16])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
def test_sums_over_many_pixel_groups(storage, k):
    """p = 2 and one constant column (the others 0): y is the mean of x over u, with x = 2^13 in the first third of the
    pixels, 2^-13 in the second and -2^13 in the last.  All products are powers of two, so a group's sums are exact,
    and the thirds are groups apart: a float32 sum over a workgroup's groups loses the second third altogether."""
    from paper_1302_2073_amd.tracker import Tracker
    width, height = 1280, 1536
    P = width * height
    U = np.zeros((P, k))
    U[:, 0] = 2.0 ** -10
    x = np.repeat([2.0 ** 13, 2.0 ** -13, -2.0 ** 13], P // 3)
    with Tracker(width, height, 1, k, storage=storage, cg_iters=1, p=2.0, mu=1e-3, delta=0.1) as t:
        t.set_launch(-1)
        t.set_state(U, np.zeros(k), None, 150)
        t.track(_tensor(x, storage))
        y = t.get_state()[1]
    assert np.isclose(y[0], 2.0 ** -3 / 3, rtol=TOL_F, atol=0)
