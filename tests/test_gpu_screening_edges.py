"""GPU: the screened interaction of prescribed pair elements at the edges of its tiles
(16 plane waves per output tile, tiles dealt over eight wavefronts, 16 pivots per group,
16 rows per slice), against numpy.

A = 1 + v^1/2 Xt v^1/2 is at least the identity: Xt carries a relative error of a few u
per row summed, the inverse of about N_G u times the condition number of A.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ng", [1, 2, 15, 16, 17, 31, 33, 48, 64, 65, 79, 96, 97, 112, 113, 127, 128])
@pytest.mark.parametrize("nv,nc", [(1, 3), (3, 4)])
def test_screening(ng, nv, nc):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_05575_amd import _lib as L
    print(f"[gpu] screening ng={ng} nv={nv} nc={nc}", flush=True)
    rng = np.random.default_rng(ng + nc)
    nk = 3
    kq = (np.arange(nk)[:, None] + np.arange(nk)[None]) % nk
    ev, ec = rng.uniform(-1, 0, (nk, nv)), rng.uniform(0.2, 1, (nk, nc))
    S1 = rng.normal(size=(nk, nk, nv, nc, ng)) + 1j * rng.normal(size=(nk, nk, nv, nc, ng))
    S2 = rng.normal(size=(nk, nk, nc, nv, ng)) + 1j * rng.normal(size=(nk, nk, nc, nv, ng))
    vs = rng.uniform(0.2, 1.0, (nk, ng))
    d = L.BseScreenDesc(nk=nk, nv=nv, nc=nc, ng=ng, inv_vc=0.05, units_per_hartree=1.0)
    t = [torch.from_numpy(np.ascontiguousarray(x)).cuda()
         for x in (ev, ec, kq.astype(np.int32), S1, S2, vs)]
    W = torch.full((nk, ng, ng), np.nan, dtype=torch.complex128, device="cuda")
    ws = torch.empty(L.bse_screening_workspace_size(d), dtype=torch.uint8, device="cuda")
    info = torch.zeros(1, dtype=torch.int32, device="cuda")
    L.bse_screening(d, *[x.data_ptr() for x in t], W.data_ptr(), ws.data_ptr(), ws.numel(),
                    info.data_ptr(), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert int(info.item()) == 0
    for q in range(nk):
        X = np.zeros((ng, ng), dtype=complex)
        for k in range(nk):
            w1 = 0.05 / (ec[kq[q, k]][None, :] - ev[k][:, None])
            w2 = 0.05 / (ec[k][:, None] - ev[kq[q, k]][None, :])
            for w, S in ((w1, S1[q, k]), (w2, S2[q, k])):
                R = S.reshape(-1, ng)
                X += R.conj().T @ (w.reshape(-1, 1) * R)
        A = np.eye(ng) + vs[q][:, None] * X * vs[q][None, :]
        ref = vs[q][:, None] * np.linalg.inv(A) * vs[q][None, :]
        tol = 2.3e-16 * (ng + 2 * nk * nv * nc + 20) * np.linalg.cond(A)
        assert np.abs(W[q].cpu().numpy() - ref).max() <= tol * np.abs(ref).max(), q
