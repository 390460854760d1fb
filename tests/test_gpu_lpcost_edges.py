"""The differentiable cost at the edges of its kernels: rows around a block and around the blocks dealt to the XCDs,
frames around the prefetch step and the passes, the widest k; outputs left out; values that are not finite."""
import ctypes as C

import numpy as np
import pytest

from test_gpu_lpcost import TOL, _oracle, _rel, _run

pytestmark = pytest.mark.gpu


def _problem(m, k, B, weighted):
    rng = np.random.default_rng([m, k, B, int(weighted)])
    U = np.linalg.qr(rng.standard_normal((m, k)))[0] if m >= k else rng.standard_normal((m, k))
    Y = rng.standard_normal((k, B))
    X = U @ Y + 0.05 * rng.standard_normal((m, B))
    w = rng.uniform(0.0, 1.0, m) if weighted else None
    return U, Y, X, w, 1e-3, 0.25, rng.uniform(0.5, 1.5, B)


# r = x - u.y carries at most (k + 1) 2^-24 (|x| + |u|.|y|), and c(r) = phi'/r at most 1.75 |r| / (r^2 + mu) <= 28 times
# that (p = 1/4, mu = 1e-3): below 1e-4 of every entry, the tolerance of the other shapes
@pytest.mark.parametrize("cost", ["lp", "log"])
@pytest.mark.parametrize("m,k,B", [(1, 1, 1), (255, 2, 2), (256, 15, 3), (257, 16, 4), (512, 16, 5), (1793, 15, 7),
                                   (2048, 3, 8), (2049, 16, 15), (2304, 15, 16), (2305, 10, 17), (700, 16, 31),
                                   (4097, 5, 32), (300, 15, 33), (511, 8, 64), (513, 16, 65)])
def test_edges(m, k, B, cost):
    U, Y, X, w, mu, p, gout = _problem(m, k, B, (m + B) % 2 == 0)
    args = (U, Y, X, w, mu, p, cost, gout)
    got, exp = _run(*args), _oracle(*args)
    errs = [_rel(a, b) for a, b in zip(got[:4], exp[:4])] + [abs(got[4] - exp[4]) / abs(exp[4])]
    assert max(errs) <= TOL, errs


@pytest.mark.parametrize("m,B", [(257, 5), (512, 17)])
def test_one_frame_that_is_not_finite_leaves_the_others(m, B):
    """A frame with an infinite coefficient, and one with an infinite upstream gradient: f, dX and dY of the other
    frames have the same bits as without them (dU and dmu sum over all frames)."""
    k, bad = 15, B // 2
    U, Y, X, w, mu, p, gout = _problem(m, k, B, True)
    clean = _run(U, Y, X, w, mu, p, "lp", gout)
    others = [b for b in range(B) if b != bad]
    Yb, gb = Y.copy(), gout.copy()
    Yb[0, bad] = np.inf
    gb[bad] = np.inf
    for args in ((U, Yb, X, w, mu, p, "lp", gout), (U, Y, X, w, mu, p, "lp", gb)):
        got = _run(*args)
        assert np.array_equal(got[0][others], clean[0][others])
        assert np.array_equal(got[2][:, others], clean[2][:, others])
        assert np.array_equal(got[3][:, others], clean[3][:, others])
    # rows past the last one of a block take no part: dmu sums positive terms, so an infinite gradient makes it
    # infinite and not NaN (dY sums terms of both signs)
    assert np.isinf(got[4])


def test_outputs_left_out():
    """Every subset of outputs of the backward: what is asked for has the same bits, nothing else is written."""
    import torch
    from paper_1302_2073_amd import _lib as L
    m, k, B = 1000, 15, 19
    U, Y, X, w, mu, p, gout = _problem(m, k, B, True)
    t = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float32, device="cuda")  # noqa: E731
    ins = [t(U), t(Y.T), t(X.T), t(w), t([mu])]
    g = t(gout)
    lib = L.lib()
    n = lib.pros_lpcost_workspace_size(m, k, B)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    ptr = lambda a: None if a is None else C.c_void_p(a.data_ptr())  # noqa: E731
    s = C.c_void_p(torch.cuda.current_stream().cuda_stream)

    def run(mask):
        outs = [torch.full(sh, 7.0, device="cuda") if mask >> i & 1 else None
                for i, sh in enumerate(((B, m), (m, k), (B, k), (1,)))]
        L.check(lib.pros_lpcost_bwd(*[ptr(a) for a in ins], m, k, B, 0, 0.25, ptr(g), *[ptr(o) for o in outs], ptr(ws),
                                    n, s))
        return [None if o is None else o.cpu().numpy() for o in outs]

    full = run(15)
    for mask in range(15):
        for a, b in zip(run(mask), full):
            assert a is None or np.array_equal(a, b)
