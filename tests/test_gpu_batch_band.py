"""GPU: the batched Cholesky factorisations and reductions over members whose orders lie on
both sides of every limit of the band reduction (432, 648, 2160, 4320: tiles of 32, 64 and
128 rows, row blocks of 64 and 128), against the plain entry points bit for bit, and the
retired choices of the tuning table, which change no bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

KEYS = ("E", "osc", "eps")


def test_uneven_members_and_retired_choices():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import bse_synth
    from bse_synth.workloads import BatchWorkload, Workload
    from paper_1904_05575_amd import _lib as L
    from paper_1904_05575_amd.batch import Batch
    common = dict(mesh=6, ng=9, coupling="full", nw=100, wmin=0.0, wmax=10.0, eta=0.05,
                  kernel_scale=1 / 16)
    bands = [(1, 2), (4, 5), (1, 3), (2, 5)]
    members = tuple(Workload(name=f"q{i}", nv=v, nc=c, seed=60 + i, q=(0.3 * i, 0.0, 0.0), **common)
                    for i, (v, c) in enumerate(bands))
    master = Workload(name="master", nv=4, nc=5, seed=59, **common)
    B = Batch(bse_synth.make_batch_inputs(BatchWorkload("uneven", members=members, master=master)),
              precision="fp64", nbranch=len(members))
    print(f"[gpu] uneven batch, orders {[m.n for m in members]}", flush=True)
    B.run()
    batched = B.results()
    B.run_sequential()
    plain = B.results()
    old = L.bse_tune_get()
    try:
        L.bse_tune_set(old + [(L.TUNE_SITES["batch_sweep"], 1 << 20, 4),
                              (L.TUNE_SITES["batch_align"], 1 << 20, 1)])
        B.captured = False  # the choices are read when the work is enqueued
        B.run()
        retired = B.results()
    finally:
        L.bse_tune_set(old)
    B.close()
    for i in range(len(members)):
        for k in KEYS:
            assert np.array_equal(batched[i][k], plain[i][k]), (i, k)
            assert np.array_equal(batched[i][k], retired[i][k]), (i, k)
