"""Re-orthonormalisation at the limits of its eigensolver: off-diagonals just above the convergence bound, and
rotations whose operands underflow."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reorthonormalised(U, y):
    from paper_1302_2073_amd.tracker import Tracker
    m, k = U.shape
    with Tracker(m, 1, 1, k) as t:
        t.set_state(U, y, None, 4)
        t.reorthonormalize()
        got, y_got, _, _ = t.get_state()
    return got, y_got


def test_off_diagonal_above_the_convergence_bound_is_rotated():
    """G = [[1, e], [e, 4 + e^2]] with 2 e^2 = 3.7e-31 of the squared diagonal: G^(1/2) (1, 0) = (1, e / 3)."""
    U = np.zeros((4, 2))
    U[0], U[1, 1] = [1.0, 2.0 ** -49], 2.0
    _, y = _reorthonormalised(U, np.array([1.0, 0.0]))
    assert np.isclose(y[0], 1.0, rtol=1e-12, atol=0)
    assert np.isclose(y[1], 2.0 ** -49 / 3, rtol=1e-12, atol=0)


def test_equal_diagonals_with_an_underflowing_off_diagonal():
    """Columns 0 and 2 have equal norms and meet only through column 1, by products of denormal entries: their
    off-diagonal, about 2^-562 after a rotation, has no square in float64.  Columns 3 to 5 keep the sweeps running."""
    U = np.zeros((8, 6))
    U[0, 0], U[1, 1], U[2, 2] = 1.0, 2.0, 1.0
    U[3, 0] = U[3, 1] = U[4, 1] = U[4, 2] = 2.0 ** -140
    U[5:, 3:] = [[1.0, 0.5, 0.3], [0.0, 1.0, 0.4], [0.0, 0.0, 1.0]]
    U = U.astype(np.float32).astype(np.float64)
    y = np.arange(1.0, 7.0)
    lam, V = np.linalg.eigh(U.T @ U)
    got, y_got = _reorthonormalised(U, y)
    assert np.allclose(got, (U @ V) / np.sqrt(lam) @ V.T, rtol=0, atol=2.0 ** -24)
    assert np.allclose(y_got, (V * np.sqrt(lam)) @ (V.T @ y), rtol=1e-12, atol=0)
