"""Launch forms changed on a live handle, the curvature schedule among them: a handle that comes back from the streamed
form runs what a fresh handle of that configuration runs, and a refused change leaves it as it was."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

W, H, C, K = 64, 60, 3, 15


def _frames(storage, width=W, height=H, n=3):
    import torch
    rng = np.random.default_rng(11)
    m = width * height * C
    U = np.linalg.qr(rng.standard_normal((m, K)))[0]
    dt = torch.float32 if storage == "f32" else torch.bfloat16
    return U, [torch.tensor(U @ rng.standard_normal(K) + 0.02 * rng.standard_normal(m), dtype=dt, device="cuda")
               for _ in range(n)]


def _result(t, U, xs):
    t.set_state(U, None, None, 7)
    stats = []
    for x in xs:
        t.track(x)
        stats.append(t.stats())
    return stats, [np.asarray(v) for v in t.get_state()], t.mask(), t.launch_info()


def _same(a, b):
    assert a[0] == b[0] and a[3] == b[3]
    assert all(np.array_equal(x, y) for x, y in zip(a[1], b[1])) and np.array_equal(a[2], b[2])


def _refused(t, *args):
    from paper_1302_2073_amd import _lib as L
    with pytest.raises(L.ProstError) as e:
        t.set_launch(*args)
    assert e.value.status == L.PROS_EUNSUPPORTED


@pytest.mark.parametrize("rows,mode", [(1, 2), (1, 3), (0, 1)])
def test_schedule_chosen_while_streamed(rows, mode):
    """float32: schedule 1 set on the streamed handle needs the wide exchange once it is resident again."""
    from paper_1302_2073_amd.tracker import Tracker
    U, xs = _frames("f32")
    with Tracker(W, H, C, K) as t, Tracker(W, H, C, K) as fresh:
        t.set_launch(-1)
        t.set_curvature(1)
        t.set_launch(rows, mode)
        fresh.set_launch(rows, mode)
        fresh.set_curvature(1)
        _same(_result(t, U, xs), _result(fresh, U, xs))
        t.set_curvature(0)
        fresh.set_curvature(0)
        _same(_result(t, U, xs), _result(fresh, U, xs))


def test_schedule_that_the_tile_kernels_do_not_have():
    """bfloat16: schedule 1 exists in the streamed form alone, so a tile is refused until schedule 0 is back."""
    from paper_1302_2073_amd.tracker import Tracker
    U, xs = _frames("bf16")
    with Tracker(W, H, C, K, storage="bf16") as t, Tracker(W, H, C, K, storage="bf16") as fresh:
        t.set_launch(-1)
        t.set_curvature(1)
        fresh.set_launch(-1)
        fresh.set_curvature(1)
        for rows in (0, 2):
            _refused(t, rows, 2)
        _same(_result(t, U, xs), _result(fresh, U, xs))
        t.set_curvature(0)
        t.set_launch(2, 2)
        with Tracker(W, H, C, K, storage="bf16") as tile:
            tile.set_launch(2, 2)
            _same(_result(t, U, xs), _result(tile, U, xs))


@pytest.mark.parametrize("width,height,forced", [(1280, 720, False), (640, 480, True)])
def test_a_refused_tile_leaves_a_streamed_handle_streamed(width, height, forced):
    """One row per thread is resident for neither frame."""
    from paper_1302_2073_amd.tracker import Tracker
    U, xs = _frames("f32", width, height, 1)
    with Tracker(width, height, C, K) as t, Tracker(width, height, C, K) as fresh:
        if forced:
            t.set_launch(-1)
            fresh.set_launch(-1)
        _refused(t, 1, 2)
        assert t.launch_info()["sync_mode"] == -1
        _same(_result(t, U, xs), _result(fresh, U, xs))
