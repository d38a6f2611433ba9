"""GPU: the pair elements of prescribed coefficients and partner tables, at the sizes
where the split into blocks changes: bands on either side of a block of five, one to
eight k-points per block (fewer where their values do not fit in LDS), odd numbers of
G and K, partners outside the sphere on both ends of the table.

An element is a sum of at most nkb products of coefficient vectors of norm one: its
rounding error is below (nkb + 4) u.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# nk, nv, nc, ng, nkb, full
SIZES = [(1, 1, 1, 1, 1, True), (3, 6, 2, 9, 7, True), (9, 4, 5, 89, 89, True),
         (10, 5, 7, 65, 33, False), (17, 1, 6, 8, 3, True), (2, 1, 1, 5, 2560, True),
         (3, 2, 11, 17, 393, False), (2, 1, 3, 33, 1280, True), (20, 4, 4, 6, 128, True),
         (19, 3, 4, 70, 129, True)]


@pytest.mark.parametrize("nk,nv,nc,ng,nkb,full", SIZES)
def test_pair_elements(nk, nv, nc, ng, nkb, full):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1904_05575_amd import _lib as L
    print(f"[gpu] pair elements nk={nk} nv={nv} nc={nc} ng={ng} nkb={nkb}", flush=True)
    rng = np.random.default_rng(nk + 10 * nv + 100 * nc + ng)
    nb = nv + nc
    C = rng.normal(size=(nk, nb, nkb)) + 1j * rng.normal(size=(nk, nb, nkb))
    C /= np.linalg.norm(C, axis=2, keepdims=True)
    tabs = [rng.integers(-nkb // 2 - 1, nkb + 2, size=(nkb, ng)).astype(np.int32) for _ in range(2)]
    P = nk * (nk + 1) // 2
    shapes = {"Mcv": (nk, nv, nc, ng), "Mvv": (P, nv, nv, ng), "Mcc": (P, nc, nc, ng),
              "Ncv": (P, nc, nv, ng), "Nvc": (P, nv, nc, ng)}
    out = {k: torch.full(s, np.nan, dtype=torch.complex128, device="cuda")
           for k, s in shapes.items()}
    Cd, kpg, mkg = (torch.from_numpy(x).cuda() for x in (C, *tabs))
    d = L.BseOrbDesc(nk=nk, nv=nv, nc=nc, ng=ng, nkb=nkb,
                     coupling=L.BSE_FULL if full else L.BSE_TDA)
    L.bse_pair_elements(d, Cd.data_ptr(), kpg.data_ptr(), mkg.data_ptr() if full else 0,
                        out["Mcv"].data_ptr(), out["Mvv"].data_ptr(), out["Mcc"].data_ptr(),
                        out["Ncv"].data_ptr() if full else 0, out["Nvc"].data_ptr() if full else 0,
                        torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    tol = (nkb + 4) * 2.3e-16

    def element(m, n, tab, conj):  # (bands at k, K) and (bands at k', K) -> (m, n, G)
        inside = (tab >= 0) & (tab < nkb)
        y = n[:, np.clip(tab, 0, nkb - 1)] * inside
        y = y.conj() if conj else y
        return np.stack([m.conj() @ y[:, :, g].T for g in range(ng)], axis=2)

    v, c = slice(0, nv), slice(nv, nb)
    p = 0
    for i in range(nk):
        for j in range(i, nk):
            want = {"Mvv": (v, v, 0), "Mcc": (c, c, 0)}
            if full:
                want |= {"Ncv": (c, v, 1), "Nvc": (v, c, 1)}
            for k, (a, b, mod) in want.items():
                ref = element(C[i, a], C[j, b], tabs[mod], mod)
                assert np.abs(out[k][p].cpu().numpy() - ref).max() <= tol, (k, i, j)
            p += 1
        ref = element(C[i, v], C[i, c], tabs[0], False)
        assert np.abs(out["Mcv"][i].cpu().numpy() - ref).max() <= tol, i
