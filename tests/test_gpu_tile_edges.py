"""Loads of the register tile at its edges: tiles that end inside a row of threads, 16-row tiles whose upper rows are
partly or wholly unused, odd pixel counts (bfloat16 halves apart, pairs that continue in the next colour plane)."""
import numpy as np
import pytest

from gpu_common import TOL_F, TOL_STEP, TOL_Y, assert_parity, compare_step
from oracle import prost_oracle as O
from synth import video as V

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("w,h,c,k,rows", [(64, 64, 1, 5, 16), (64, 65, 1, 5, 16), (80, 60, 1, 5, 16), (86, 83, 1, 4, 16),
                                          (128, 64, 1, 5, 16), (37, 29, 3, 3, 4), (37, 29, 3, 15, 8), (51, 41, 4, 15, 8),
                                          (7, 3, 2, 2, 2), (131, 129, 3, 12, 8)])
def test_step_on_partial_tiles(w, h, c, k, rows, storage):
    """One frame against the float64 oracle, float32 at the parity bar; in bfloat16 the frame is rounded first and a
    stored entry of U lies within a unit in the last place (2^-8) of the largest.  Two frames in one launch give the
    bits of two launches."""
    from paper_1302_2073_amd import Tracker
    from paper_1302_2073_amd.tracker import bf16_bits, bf16_to_f64
    prm = O.Params(w, h, c, k=k, i_init=5)
    rng = np.random.default_rng([w, h, c, k])
    m = w * h * c
    U = V.initial_subspace(m, k, 3)
    scale = np.sqrt(m / k)
    xs = [U @ (scale * rng.uniform(0.2, 0.5, k)) + 0.02 * rng.standard_normal(m) for _ in range(2)]
    xs = [x.astype(np.float32).astype(np.float64) if storage == "f32" else bf16_to_f64(bf16_bits(x)) for x in xs]
    labels = (rng.uniform(size=w * h) < 0.2).astype(np.uint8)
    start = O.State(U, scale * rng.uniform(0.2, 0.5, k), labels, O.median3x3(labels, h, w), 3)
    with Tracker(w, h, c, k, storage=storage, i_init=5) as t:
        t.set_launch(rows)
        rep = compare_step(t, prm, start, xs[0], storage=storage)
        if storage == "f32":
            assert_parity(rep)
        else:
            assert rep["y_rel"] <= TOL_Y and rep["f_rel"] <= TOL_F and rep["theta_rel"] <= TOL_STEP
            assert rep["lab_mismatch_outside_band"] == 0 and rep["U_elem"] <= 2.0 ** -8
        t.track(xs[1].astype(np.float32) if storage == "f32" else bf16_bits(xs[1]))
        want = t.get_state()
        import torch
        dev = [torch.from_numpy(x.astype(np.float32)).cuda() if storage == "f32" else
               torch.from_numpy(bf16_bits(x).view(np.int16)).cuda().view(torch.bfloat16) for x in xs]
        t.set_state(start.U, start.y, start.labels, start.n)
        t.track_many(dev)
        assert all(np.array_equal(a, b) for a, b in zip(want, t.get_state()))
