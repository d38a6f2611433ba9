"""GPU: the band reduction of matrices far from one in size, and of matrices whose panels
are not zero but negligible.

Eigenvalues within 20 sqrt(n) u ||A||_2 (as for any product of this many reflectors).
"""
import numpy as np
import pytest

from test_gpu_band import _random, _solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size", [1e-139, 1e-150, 1e-157, 1e-160, 1e-200])
@pytest.mark.parametrize("cut", [96, 90])
def test_couplings_near_underflow(cut, size):
    """Two blocks joined by elements whose squares leave the normal range, at the end of a
    panel and inside one: they change no eigenvalue, and the squared norms of such columns
    must not be divided by."""
    n = 220
    print(f"[gpu] band reduction, blocks cut at {cut} joined by {size:g}", flush=True)
    a = np.zeros((n, n), dtype=complex)
    a[:cut, :cut], a[cut:, cut:] = _random(cut, 3), _random(n - cut, 4)
    x = size * (np.random.default_rng(5).normal(size=(n - cut, cut)) + 0.5j)
    a[cut:, :cut], a[:cut, cut:] = x, x.conj().T
    E, osc = _solve(a, np.ones(n) + 0j)
    E0 = np.sort(np.concatenate([np.linalg.eigvalsh(a[:cut, :cut]),
                                 np.linalg.eigvalsh(a[cut:, cut:])]))
    assert np.abs(E - E0).max() <= 20.0 * np.sqrt(n) * np.finfo(float).eps * np.abs(E0).max()
    assert abs(osc.sum() / n - 1) <= 1e-10


@pytest.mark.parametrize("scale", [1e-135, 1e-120, 1e120, 1e150])
def test_scaled_matrices(scale):
    """The eigenvalues scale with the matrix while the squares of its elements are well
    inside the range of double precision."""
    n = 220
    print(f"[gpu] band reduction, elements of {scale:g}", flush=True)
    a = _random(n, 6)
    E, osc = _solve(a * scale, np.ones(n) + 0j)
    E0 = np.linalg.eigvalsh(a)
    assert np.abs(E / scale - E0).max() <= 20.0 * np.sqrt(n) * np.finfo(float).eps * np.abs(E0).max()
    assert abs(osc.sum() / n - 1) <= 1e-10
