"""GPU: the reduction to band form at the orders where its tiles change (128 rows x 64
columns while more than 2048 rows are left), with ragged last tiles.

Eigenvalues within 1e-12 n max|A| of LAPACK's (a Householder-type reduction is backward
stable to a small multiple of n u ||A||), and the probe's weights add up to its norm
(unitary transformations, 1e-10 relative for n of them).
"""
import numpy as np
import pytest

from test_gpu_band import _solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2065, 2129, 2200])
def test_tall_tiles(n):
    print(f"[gpu] band reduction, tall tiles, n={n}", flush=True)
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
    a = x + x.conj().T
    p = rng.normal(size=n) + 1j * rng.normal(size=n)
    E, osc = _solve(a, p)
    assert np.abs(E - np.linalg.eigvalsh(a)).max() <= 1e-12 * n * np.abs(a).max()
    assert abs(osc.sum() / np.vdot(p, p).real - 1) <= 1e-10
