"""Gang exchanges at the edges of their layouts: gangs around the group count, the rows a wavefront gathers and the
largest residents, and value counts below, at and above the 16 lanes of a row (k = 1, 2, 14, 15, 16)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(t, U, xs, rows, mode):
    t.set_launch(rows, mode)
    t.set_state(U, None, None, 7)
    out = []
    for x in xs:
        t.track(x)
        out.append(t.stats())
    many = t.get_state()
    return out, many, t.mask(), t.launch_info()["workgroups"]


@pytest.mark.parametrize("k", [1, 2, 14, 15, 16])
@pytest.mark.parametrize("width,height", [(32, 17), (64, 56), (64, 57), (64, 72), (128, 130), (512, 65), (512, 129),
                                          (512, 255)])
def test_tagged_exchanges_agree_with_the_counter(width, height, k):
    """Exchanges 2 and 3 against exchange 0 (plain float64 sums): the first cost is one sum of the same workgroup
    partials, of which the tags take 8 of 52 mantissa bits at most twice and the order moves the last few: 2^-42.
    What follows from it is float32 work on sums that may differ in the last float32 place."""
    import torch
    from paper_1302_2073_amd.tracker import Tracker
    m = width * height
    rng = np.random.default_rng([width, height, k])
    U = np.linalg.qr(rng.standard_normal((m, k)))[0]
    xs = [torch.tensor(U @ rng.standard_normal(k) + 0.02 * rng.standard_normal(m), dtype=torch.float32, device="cuda")
          for _ in range(3)]
    with Tracker(width, height, 1, k) as t:
        want, state, mask, gang = _run(t, U, xs, 1, 0)
        assert gang == -(-m // 512)
        for mode in (2, 3):
            got, state2, mask2, _ = _run(t, U, xs, 1, mode)
            for a, b in zip(want, got):
                assert a["cg_steps"] == b["cg_steps"] and a["updated"] == b["updated"]
                assert np.allclose(b["f"], a["f"], rtol=1e-6, atol=0)
                assert np.isclose(b["theta"], a["theta"], rtol=1e-5, atol=0)
            assert abs(got[0]["f"][0] - want[0]["f"][0]) <= 2.0 ** -42 * want[0]["f"][0]
            assert np.abs(state2[0] - state[0]).max() <= 1e-6 and state2[3] == state[3]
            again, state3, mask3, _ = _run(t, U, xs, 1, mode)     # deterministic
            assert all(np.array_equal(p, q) for p, q in zip(state2, state3)) and np.array_equal(mask2, mask3)
            t.set_state(U, None, None, 7)                         # several frames in one launch: the same bits
            t.track_many(xs)
            assert t.stats()["f"] == got[-1]["f"]
            assert all(np.array_equal(p, q) for p, q in zip(state2, t.get_state()))
            assert np.array_equal(t.mask(), mask2)
