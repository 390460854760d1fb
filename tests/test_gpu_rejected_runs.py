"""Long runs of rejected frames between two good ones.  A rejected frame takes one exchange and leaves the slots of the
others with the tags of the last good frame, which repeat after 256 exchanges: the frame after the run must not take
those for its own."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

W, H, C, K, J = 64, 60, 3, 5, 5


def _frames(storage):
    import torch
    rng = np.random.default_rng(5)
    m = W * H * C
    U = np.linalg.qr(rng.standard_normal((m, K)))[0]
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    good = [torch.tensor(U @ rng.standard_normal(K) + 0.02 * rng.standard_normal(m), dtype=dt, device="cuda")
            for _ in range(2)]
    nan = good[0].clone()
    nan[m // 2] = float("nan")
    return U, good, nan


def _run(t, U, frames, many):
    t.set_state(U, None, None, 7)
    if many:
        t.track_many(frames)
    else:
        for x in frames:
            t.track(x)
    t.sync()
    s = t.stats()
    return s, [np.asarray(v) for v in t.get_state()], t.mask()


# a good frame takes 2 J + 1 exchanges (J + 1 where H is reduced with the gradient); its last one meets its own tags, or
# those of the frame before it in the other slot set, after this many rejected frames
PLAIN = [256 - (2 * J + 1), 256 - 2 * (2 * J + 1)]
WIDE = [256 - (J + 1)]


@pytest.mark.parametrize("many", [False, True])
@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("run", PLAIN)
def test_plain_frames(run, mode, storage, many):
    from paper_1302_2073_amd.tracker import Tracker
    U, good, nan = _frames(storage)
    rows = 1 if storage == "f32" else 2
    with Tracker(W, H, C, K, storage=storage, cg_iters=J) as t, Tracker(W, H, C, K, storage=storage, cg_iters=J) as want:
        for h in (t, want):
            h.set_launch(rows, mode)
        a = _run(t, U, [good[0], good[1]] + [nan] * run + [good[0]], many)
        b = _run(want, U, [good[0], good[1], good[0]], many)
    assert a[0] == b[0]
    assert all(np.array_equal(x, y) for x, y in zip(a[1], b[1])) and np.array_equal(a[2], b[2])


@pytest.mark.parametrize("solver", ["cg", "irls"])
@pytest.mark.parametrize("mode", [1, 2, 3])
@pytest.mark.parametrize("run", WIDE)
def test_frames_with_the_wide_exchange(run, mode, solver):
    from paper_1302_2073_amd.tracker import Tracker
    U, good, nan = _frames("f32")
    with Tracker(W, H, C, K, cg_iters=J, ysolve=solver) as t, Tracker(W, H, C, K, cg_iters=J, ysolve=solver) as want:
        for h in (t, want):
            h.set_launch(1, mode)
            if solver == "cg":
                h.set_curvature(1)
        a = _run(t, U, [good[0], good[1]] + [nan] * run + [good[0]], False)
        b = _run(want, U, [good[0], good[1], good[0]], False)
    assert a[0] == b[0]
    assert all(np.array_equal(x, y) for x, y in zip(a[1], b[1])) and np.array_equal(a[2], b[2])
