"""GPU: backward error of the Cholesky factorisation A - B = U^H U where a diagonal block
U11 is ill-conditioned (condition up to 10^6.2), through the energies of the full solve.

E^2 are the eigenvalues of S = U (A+B) U^H.  The factorisation is backward stable to a
few n u ||A-B|| whatever the condition of its blocks, and LAPACK's is too, so E^2 agree
within 20 sqrt(n) u ||S||_2 as the errors of n columns add up like a random walk, once
the reduction's own error of the same size is counted (a panel row whose error carries
cond(U11) is 10 to 1000 times off).
"""
import numpy as np
import pytest

from test_gpu_cholesky import _definite, _solve

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [96, 200])
@pytest.mark.parametrize("k", [4.0, 6.0, 6.2])
@pytest.mark.parametrize("j0", [0, 32])
def test_ill_conditioned_diagonal_block(n, k, j0):
    print(f"[gpu] cholesky, condition 10^{k} in panel {j0} of {n}", flush=True)
    rng = np.random.default_rng(int(10 * k) + n + j0)
    r = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    # A - B = F^H F, whose 32 columns from j0 are nearly dependent; the others reach into
    # their span.  The smallest eigenvalue stays some 10^-2k ||S||, above the n u ||S|| at
    # which the solve reports a non-positive one.
    q, _ = np.linalg.qr(r(n, n))
    w, _ = np.linalg.qr(r(32, 32))
    rest = q[:, 32:] + q[:, :32] @ r(32, n - 32) * (0.2 / np.sqrt(32))
    panel = (q[:, :32] * 10.0 ** (-k * np.arange(32) / 31)) @ w
    f = np.concatenate([rest[:, :j0], panel, rest[:, j0:]], axis=1)
    m = f.conj().T @ f
    m = 0.5 * (m + m.conj().T)
    p = _definite(n, rng)
    p = 0.5 * (p + p.conj().T)
    E = _solve(p, m, 0)
    u = np.linalg.cholesky(m).conj().T
    s = u @ p @ u.conj().T
    mu = np.linalg.eigvalsh(0.5 * (s + s.conj().T))
    err = np.abs(E ** 2 - mu).max() / mu.max()
    print(f"[gpu] error {err:.1e}", flush=True)
    assert err <= 20.0 * np.sqrt(n) * np.finfo(float).eps
