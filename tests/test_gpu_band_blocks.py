"""GPU: the band reduction of matrices that fall into blocks or narrow bands, whose panels
are dependent and zero past a few rows: against LAPACK, over extents on both sides of 64
rows and of the row blocks of the panel kernels (64 rows, 128 beyond 4096), and its time.

Eigenvalues within 20 sqrt(n) u ||A||_2 (as for any product of this many reflectors).
"""
import numpy as np
import pytest

from test_gpu_band import _random, _solve

pytestmark = pytest.mark.gpu


def _blocks(n, size):
    a = np.zeros((n, n), dtype=complex)
    for j in range(0, n, size):
        m = min(size, n - j)
        a[j:j + m, j:j + m] = _random(m, n + j)
    return a


def _banded(n, width):
    a = _random(n, n)
    i = np.arange(n)
    return np.where(np.abs(i[:, None] - i[None, :]) <= width, a, 0.0)


@pytest.mark.parametrize("n,make,size", [
    (150, _blocks, 1), (333, _blocks, 12), (400, _blocks, 17), (500, _blocks, 60),
    (500, _blocks, 64), (501, _blocks, 70), (700, _blocks, 150), (400, _banded, 1),
    (401, _banded, 5), (400, _banded, 15), (400, _banded, 16), (401, _banded, 40),
    (4400, _blocks, 40), (4400, _banded, 1)])
def test_blocks_and_bands(n, make, size):
    print(f"[gpu] band reduction, {make.__name__} {size}, n={n}", flush=True)
    a = make(n, size)
    p = np.random.default_rng(n).normal(size=n) + 0.5j
    E, osc = _solve(a, p)
    if make is _blocks:
        E0 = np.sort(np.concatenate([np.linalg.eigvalsh(a[j:j + size, j:j + size])
                                     for j in range(0, n, size)]))
    elif size == 1:
        from scipy.linalg import eigvalsh_tridiagonal
        E0 = eigvalsh_tridiagonal(np.diag(a).real, np.abs(np.diag(a, -1)))
    else:
        E0 = np.linalg.eigvalsh(a)
    assert np.abs(E - E0).max() <= 20.0 * np.sqrt(n) * np.finfo(float).eps * np.abs(E0).max()
    assert abs(osc.sum() / np.vdot(p, p).real - 1) <= 1e-10


@pytest.mark.parametrize("n", [1000, 2000])
def test_a_tridiagonal_matrix_costs_no_more_than_a_dense_one(n):
    """Dependent panels of few rows, in every panel: at most one and a half times the
    time of the same order with dense panels (best of five each)."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_05575_amd import _lib as L
    print(f"[gpu] time of a tridiagonal matrix, n={n}", flush=True)
    d = L.BseDesc(nk=1, nv=1, nc=n, ng=9, coupling=L.BSE_TDA, type=L.BSE_SINGLET,
                  prec=L.BSE_PREC_FP64, split_terms=0, kappa=1.0, scissor=0.0, ld=n)
    ws = torch.empty(L.bse_workspace_size(d, L.BSE_STAGE_SOLVE), dtype=torch.uint8, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    E = torch.empty(n, dtype=torch.float64, device="cuda")
    osc, P = torch.empty_like(E), torch.ones(n, dtype=torch.complex128, device="cuda")

    def best(a):
        H, t = torch.from_numpy(np.ascontiguousarray(a.T)).cuda(), []
        for _ in range(5):
            h = H.clone()
            e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            e[0].record()
            L.bse_solve(d, h.data_ptr(), 0, E.data_ptr(), 0, 0, n, P.data_ptr(), osc.data_ptr(),
                        ws.data_ptr(), ws.numel(), info.data_ptr(),
                        torch.cuda.current_stream().cuda_stream)
            e[1].record()
            torch.cuda.synchronize()
            t.append(e[0].elapsed_time(e[1]))
        assert int(info.item()) == 0
        return min(t)

    dense, narrow = best(_random(n, 1)), best(_banded(n, 1))
    print(f"[gpu] {dense:.2f} ms dense, {narrow:.2f} ms tridiagonal", flush=True)
    assert narrow <= 1.5 * dense
