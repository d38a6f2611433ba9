"""GPU: backward error of the band reduction on panels that are nearly dependent but
still take the Gram route: condition numbers of 10^4 to 10^7 and relative pivots down to
the threshold of 1e-11, in both branches of its second pass, and on smooth kernels, whose
first panels leave that route.

The reduction is a product of n / 16 block reflectors and about n^2 / 16 reflectors of
the chase.  Each commits a few u ||A||, and they add up like a random walk over the n
columns that each passes: eigenvalues within 20 sqrt(n) u ||A||_2 of LAPACK's, whose own
error is smaller (a reduction whose panel residual grows as u cond(P) is 10 to 1000 times
above that here).
"""
import numpy as np
import pytest

from test_gpu_band import _random, _solve

pytestmark = pytest.mark.gpu

N = 400


def _geometric(rng, k):
    """First panel: singular values falling geometrically to 10^-k, random vectors."""
    r = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    u, _ = np.linalg.qr(r(N - 16, 16))
    v, _ = np.linalg.qr(r(16, 16))
    return np.sqrt(N) * (u * 10.0 ** (-k * np.arange(16) / 15)) @ v.conj().T


def _dependent(rng, eps):
    """First panel: column 1 is column 0 up to eps noise, and the other columns lie
    largely along that noise."""
    r = lambda *s: rng.normal(size=s) + 1j * rng.normal(size=s)  # noqa: E731
    p, noise = r(N - 16, 16), r(N - 16)
    p[:, 1] = p[:, 0] + eps * noise
    p[:, 2:] += 3.0 * noise[:, None]
    return p


def _growing(rng, scale):
    """First panel: unit columns whose triangular factor has an inverse that doubles from
    column to column, with no small pivot early on."""
    q, _ = np.linalg.qr(rng.normal(size=(N - 16, 16)) + 1j * rng.normal(size=(N - 16, 16)))
    t = (np.eye(16) - np.triu(np.ones((16, 16)), 1)) * (scale ** np.arange(16))[:, None]
    return q @ t * (np.sqrt(N) / np.linalg.norm(t, axis=0))


def _matrix(kind, x):
    rng = np.random.default_rng(17)
    if kind == "smooth":
        g = np.linspace(0.0, 1.0, N)
        return np.exp(-((g[:, None] - g[None, :]) / x) ** 2) + np.diag(1 + np.cos(7 * g)) + 0j
    a = _random(N, 23)
    a[16:, :16] = {"geometric": _geometric, "dependent": _dependent, "growing": _growing}[kind](rng, x)
    a[:16, 16:] = a[16:, :16].conj().T
    return a


@pytest.mark.parametrize("kind,x", [("geometric", 4.0), ("geometric", 5.5), ("geometric", 6.0),
                                    ("geometric", 6.5), ("dependent", 1e-2), ("dependent", 1e-4),
                                    ("dependent", 1e-5), ("dependent", 5e-6), ("dependent", 4e-6),
                                    ("growing", 1.0), ("growing", 0.8), ("growing", 0.7),
                                    ("growing", 0.6), ("smooth", 0.3), ("smooth", 0.1)])
def test_nearly_dependent_panels(kind, x):
    print(f"[gpu] band reduction, {kind} panel {x:g}", flush=True)
    a = _matrix(kind, x)
    p = np.ones(N) + 0.5j
    E, _ = _solve(a, p)
    E0 = np.linalg.eigvalsh(a)
    err = np.abs(E - E0).max() / np.abs(E0).max()
    print(f"[gpu] error {err:.1e}", flush=True)
    assert err <= 20.0 * np.sqrt(N) * np.finfo(float).eps
