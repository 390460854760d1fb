"""Re-orthonormalisation at the edges of its kernels: every subspace dimension class (odd ones are padded to even in
the eigensolver), row counts around the wavefront tiles, both storage types, near-orthonormal and badly scaled U."""
import numpy as np
import pytest

from oracle import prost_oracle as O

pytestmark = pytest.mark.gpu


def _stored(U, storage):
    from paper_1302_2073_amd.tracker import bf16_bits, bf16_to_f64
    return U.astype(np.float32).astype(np.float64) if storage == "f32" else bf16_to_f64(bf16_bits(U))


@pytest.mark.parametrize("storage", ["f32", "bf16"])
@pytest.mark.parametrize("width,height,channels,k", [(1, 1, 1, 1), (2, 1, 1, 2), (17, 1, 1, 3), (31, 1, 1, 4),
                                                     (11, 3, 1, 5), (127, 1, 1, 8), (43, 3, 1, 11), (86, 3, 1, 15),
                                                     (16, 16, 1, 16), (123, 47, 3, 15), (320, 240, 3, 10)])
def test_reorthonormalisation_matches_the_polar_factor(width, height, channels, k, storage):
    """U is the float64 polar factor rounded once: within half a unit of the storage type (and the 2^-40 that float64
    sums over the rows may move it), y = G^(1/2) y to float64 rounding."""
    from paper_1302_2073_amd.tracker import Tracker
    m = width * height * channels
    rng = np.random.default_rng([m, k])
    Q = np.linalg.qr(rng.standard_normal((m, k)))[0]
    for spread in (1e-3, 0.5):
        U = _stored(Q @ (np.eye(k) + spread * rng.standard_normal((k, k)) / k), storage)
        y = rng.standard_normal(k)
        lam, V = np.linalg.eigh(U.T @ U)
        want, y_want = (U @ V) / np.sqrt(lam) @ V.T, (V * np.sqrt(lam)) @ (V.T @ y)
        assert np.allclose(want, O.lowdin(U)[0], atol=1e-11)
        with Tracker(width, height, channels, k, storage=storage) as t:
            t.set_state(U, y, None, 4)
            t.reorthonormalize()
            got, y_got, _, n = t.get_state()
        assert n == 4
        bits = 24 if storage == "f32" else 8
        unit = 2.0 ** (np.floor(np.log2(np.maximum(np.abs(want), 1e-30))) + 1 - bits)
        assert np.all(np.abs(got - want) <= 0.5 * unit * (1.0 + 2.0 ** -15) + 1e-12)
        assert np.allclose(y_got, y_want, rtol=0, atol=1e-11 * np.abs(y_want).max())
