"""GPU: the choice of four real products per complex one reaches every tile edge of the
complex GEMM.  The exchange term of coefficients whose imaginary parts are 1e-10 of their
real ones: im V = sum_G v (ar bi - ai br) has products of that size only, and four real
products sum just these.

Error bound: N_G products and sums and a few more roundings, (N_G + 8) u times the sum
of the products' moduli, twice for the reference's own.  (Three products carry u |a| |b|,
10^10 times as much.)
"""
import numpy as np
import pytest

from tests._cache import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile", [16, 32, 64])
@pytest.mark.parametrize("name", ["small_full_k3_v3c4_g27", "tda_q0_k4_v2c3_g59"])
def test_four_products_on_every_edge(name, tile):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_05575_amd import _lib as L
    from paper_1904_05575_amd.bse import Problem
    print(f"[gpu] {name} four products, tile {tile}", flush=True)
    d = dict(inputs(name))
    M = d["Mcv"].real + 1e-10j * d["Mcv"].imag
    d["Mcv"] = M
    P = Problem(d, bse_type="rpa")  # no direct term
    old = L.bse_tune_get()
    try:
        L.bse_tune_set([(L.TUNE_SITES["gemm_exchange"], 1 << 20, tile),
                        (L.TUNE_SITES["gemm_products"], 1 << 20, 4)])
        H0, _ = P.build()
        P.check_info()
    finally:
        L.bse_tune_set(old)
    got = H0.T.cpu().numpy().imag
    v = P.t["vbar"].cpu().numpy() * (4.0 if P.full else 2.0) * P.kappa
    a, b = M.real, M.imag
    ref = (a * v) @ b.T - (b * v) @ a.T
    size = np.abs(a * v) @ np.abs(b).T + np.abs(b * v) @ np.abs(a).T
    bound = 2.0 * (P.ng + 8) * (np.finfo(float).eps / 2) * size
    assert (np.abs(got - ref) <= bound).all()
