"""GPU: the blocked Cholesky factorisation A - B = U^H U inside the full solve, on
prescribed matrices at the edges of its panels (32 columns, factored in pairs, 64
columns of the panel row per block), against LAPACK through the solve's energies,
and the column it reports when A - B is not positive definite.

The energies are the square roots of the eigenvalues of U (A+B) U^H; with both
matrices' condition numbers near 20 they carry a relative error of about n u
times that: 1e-12 n is two orders above it.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _solve(apb, amb, expect):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_05575_amd import _lib as L
    n = apb.shape[0]
    d = L.BseDesc(nk=1, nv=1, nc=n, ng=9, coupling=L.BSE_FULL, type=L.BSE_SINGLET,
                  prec=L.BSE_PREC_FP64, split_terms=0, kappa=1.0, scissor=0.0, ld=n)
    H0, H1 = (torch.from_numpy(np.ascontiguousarray(m.T)).cuda() for m in (apb, amb))
    E = torch.empty(n, dtype=torch.float64, device="cuda")
    ws = torch.empty(L.bse_workspace_size(d, L.BSE_STAGE_SOLVE), dtype=torch.uint8, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    probe, osc = torch.ones(n, dtype=torch.complex128, device="cuda"), torch.empty_like(E)
    L.bse_solve(d, H0.data_ptr(), H1.data_ptr(), E.data_ptr(), 0, 0, n, probe.data_ptr(),
                osc.data_ptr(), ws.data_ptr(), ws.numel(), info.data_ptr(),
                torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert int(info.item()) == expect
    return E.cpu().numpy()


def _definite(n, rng):
    x = rng.normal(size=(n, n)) + 1j * rng.normal(size=(n, n))
    q, _ = np.linalg.qr(x)
    return (q * rng.uniform(1.0, 20.0, n)) @ q.conj().T


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 95, 96, 97, 128, 129, 161, 225])
def test_energies(n):
    print(f"[gpu] cholesky n={n}", flush=True)
    rng = np.random.default_rng(n)
    p, m = _definite(n, rng), _definite(n, rng)
    E = _solve(0.5 * (p + p.conj().T), 0.5 * (m + m.conj().T), 0)
    u = np.linalg.cholesky(0.5 * (m + m.conj().T)).conj().T
    s = u @ p @ u.conj().T
    ref = np.sqrt(np.linalg.eigvalsh(0.5 * (s + s.conj().T)))
    assert np.abs(E / ref - 1).max() <= 1e-12 * n


@pytest.mark.parametrize("n,col", [(1, 0), (40, 0), (40, 31), (40, 32), (40, 39), (100, 63),
                                   (100, 64), (100, 97)])
def test_first_column_that_fails(n, col):
    print(f"[gpu] cholesky, not positive definite at {col} of {n}", flush=True)
    d = np.full(n, 2.0)
    d[col:] = -1.0          # every later pivot is bad too: the first one is reported
    _solve(np.eye(n, dtype=complex), np.diag(d).astype(complex), col + 1)


@pytest.mark.parametrize("bad", [0, 1, 3])
def test_failing_member_of_a_batch(bad):
    """One member's A - B is not positive definite: its status says so and the
    other members' energies are those of the batch without it failing, bit for bit."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from bse_synth import BATCHES, make_batch_inputs
    from paper_1904_05575_amd.batch import Batch
    print(f"[gpu] batch with member {bad} failing", flush=True)
    B = Batch(make_batch_inputs(BATCHES["batch4_k2_g15"]), precision="fp64", nbranch=4)
    B.run()
    good = [r["E"].copy() for r in B.results()]
    B.t[bad]["eps_c"] = B.t[bad]["eps_c"] - 100.0  # conduction far below valence
    B.inputs[bad].eps_c = B.t[bad]["eps_c"].data_ptr()
    B.captured = False
    B.run()
    torch.cuda.synchronize()
    info = B.info.cpu().numpy()
    assert info[bad] != 0 and np.count_nonzero(info) == 1
    for i, t in enumerate(B.t):
        assert i == bad or np.array_equal(t["E"].cpu().numpy(), good[i])
    B.close()
