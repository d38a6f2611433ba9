"""GPU: the Lorentzian sums at the edges of their split (16 levels per row of lanes, 128
per step; one, two or four frequencies per lane, 4 lanes of frequencies per wavefront)
and for energies whose squares leave the range of double precision.

Each term is within about 20 u of the sum of its two fractions' magnitudes, and the sum
of n of them adds at most n u of the same: the bound is (n + 30) u times the sum of the
magnitudes.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _call(E, osc, t, om, eta, pref):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_05575_amd import _lib as L
    Ed, od, td, wd = (torch.from_numpy(x).cuda() for x in (E, osc, t, om))
    nd, n, nw = t.shape[0], len(E), len(om)
    eps = torch.empty(nw, dtype=torch.complex128, device="cuda")
    ten = torch.empty((nw, nd, nd), dtype=torch.complex128, device="cuda")
    s = torch.cuda.current_stream().cuda_stream
    L.bse_spectrum(n, Ed.data_ptr(), od.data_ptr(), pref, eta, nw, wd.data_ptr(), eps.data_ptr(), s)
    L.bse_dielectric_tensor(n, Ed.data_ptr(), nd, td.data_ptr(), n, pref, eta, nw, wd.data_ptr(),
                            ten.data_ptr(), s)
    torch.cuda.synchronize()
    return eps.cpu().numpy(), ten.cpu().numpy()


def _check(E, osc, t, om, eta, pref):
    eps, ten = _call(E, osc, t, om, eta, pref)
    nd, tol = t.shape[0], (len(E) + 30) * 2.3e-16 * abs(pref)
    w = om[:, None]
    g1, g2 = 1 / (w - E + 1j * eta), 1 / (w + E + 1j * eta)
    g, ga = g1 - g2, np.abs(g1) + np.abs(g2)
    err = np.abs(eps - (1 - pref * (osc * g).sum(1)))
    assert np.all(err <= tol * (np.abs(osc) * ga).sum(1) + 2.3e-16)
    for a in range(nd):
        for b in range(nd):
            ref = (a == b) - pref * (t[a].conj() * t[b] * g).sum(1)
            err = np.abs(ten[:, a, b] - ref)
            assert np.all(err <= tol * (np.abs(t[a] * t[b]) * ga).sum(1) + 2.3e-16), (a, b)


@pytest.mark.parametrize("nd", [1, 2, 3])
@pytest.mark.parametrize("n,nw", [(1, 1), (15, 5), (17, 1535), (128, 1537), (129, 3071), (1000, 3073)])
def test_split(n, nw, nd):
    print(f"[gpu] lorentz n={n} nw={nw} nd={nd}", flush=True)
    rng = np.random.default_rng(n + nd)
    E = np.sort(rng.uniform(0.05, 1.0, n))
    t = rng.normal(size=(nd, n)) + 1j * rng.normal(size=(nd, n))
    _check(E, rng.uniform(0, 1, n), t, np.linspace(-0.2, 1.2, nw), 3e-3, 0.7)


def test_range():
    """Levels whose |d|^2 overflows or underflows, among ordinary ones."""
    print("[gpu] lorentz range", flush=True)
    rng = np.random.default_rng(3)
    E = rng.uniform(0.05, 1.0, 70)
    E[[3, 20, 69]] = [1e120, 1e-120, 0.0]
    t = rng.normal(size=(2, 70)) + 1j * rng.normal(size=(2, 70))
    om = np.array([0.0, 1e-120, 0.3, E[7], 1e110])
    for eta in (1e-3, 1e-90):
        _check(E, rng.uniform(0, 1, 70), t, om, eta, 0.5)
