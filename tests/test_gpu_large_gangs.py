"""Gangs of more than one workgroup per compute unit, which pros_set_launch accepts as long as they are resident, and
buffered sequences on them (the sequence form holds fewer of its workgroups)."""
import numpy as np
import pytest

from gpu_common import TOL_F, TOL_Y

pytestmark = pytest.mark.gpu


def _frames(m, k, storage, n):
    import torch
    rng = np.random.default_rng([m, k])
    A = rng.standard_normal((m, k))
    U = A @ np.linalg.inv(np.linalg.cholesky(A.T @ A).T)
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    return U, [torch.tensor(U @ rng.standard_normal(k) + 0.02 * rng.standard_normal(m), dtype=dt, device="cuda")
               for _ in range(n)]


@pytest.mark.parametrize("width,height,k,storage,rows,gang", [(640, 480, 10, "f32", 4, 451), (640, 640, 6, "bf16", 8, 301)])
def test_sequence_of_a_gang_that_its_kernel_does_not_hold(width, height, k, storage, rows, gang):
    """The frame kernel holds two workgroups per compute unit here, the sequence form one."""
    from paper_1302_2073_amd.tracker import Tracker
    U, xs = _frames(width * height * 3, k, storage, 3)
    out = []
    for many in (False, True):
        with Tracker(width, height, 3, k, storage=storage) as t:
            t.set_launch(rows, 2)
            assert t.launch_info()["workgroups"] == gang
            t.set_state(U, None, None, 7)
            if many:
                t.track_many(xs)
            else:
                for x in xs:
                    t.track(x)
            out.append((t.stats(), t.get_state(), t.mask()))
    assert out[0][0] == out[1][0] and np.array_equal(out[0][2], out[1][2])
    assert all(np.array_equal(a, b) for a, b in zip(out[0][1], out[1][1]))


@pytest.mark.parametrize("width,height,k,storage,rows,gang,kw", [
    (640, 480, 15, "f32", 4, 451, {}), (480, 320, 5, "f32", 1, 904, {}), (480, 320, 4, "f32", 1, 904, {}),
    (640, 320, 11, "f32", 2, 601, {}), (640, 640, 3, "f32", 4, 601, {}),
    (400, 300, 15, "f32", 2, 352, {"ysolve": "irls"}), (640, 640, 3, "f32", 8, 301, {"preprocess": 1}),
    (640, 320, 12, "bf16", 2, 603, {}), (640, 640, 2, "bf16", 4, 601, {}), (640, 640, 12, "bf16", 8, 301, {}),
    (1280, 640, 3, "bf16", 16, 301, {}), (640, 640, 11, "bf16", 8, 301, {"preprocess": 1})])
def test_register_limited_tiles(width, height, k, storage, rows, gang, kw):
    """Gangs that only the kernels with a register limit hold, against the handle's own choice: the same frames with
    the sums split over other workgroups."""
    from paper_1302_2073_amd.tracker import Tracker
    U, xs = _frames(width * height * 3, k, storage, 2)
    out = []
    for forced in (False, True):
        with Tracker(width, height, 3, k, storage=storage, **kw) as t:
            if forced:
                t.set_launch(rows, 2)
                assert t.launch_info()["workgroups"] == gang
            t.set_state(U, None, None, 7)
            for x in xs:
                t.track(x)
            out.append((t.stats(), t.get_state()))
    (a, sa), (b, sb) = out
    assert a["cg_steps"] == b["cg_steps"] and np.allclose(a["f"], b["f"], rtol=TOL_F, atol=0)
    assert np.linalg.norm(sa[1] - sb[1]) <= TOL_Y * np.linalg.norm(sa[1])
    assert np.linalg.norm(sa[0] - sb[0]) <= (1e-5 if storage == "f32" else 2.0 ** -8) * np.linalg.norm(sa[0])
    assert np.mean(sa[2] != sb[2]) < 1e-3
