"""The reconstruction and its transpose at counts of rows, moments and energies on both sides of what their kernels
take at once (four rows a thread, 16 energies to 256 a workgroup, tiles of 64 moments in chains of 16; groups of 8
moments shared by 1 to 256 threads), and for many rows or few energies in a time that grows with the work.
Bar: normwise 1e-10, as for the kernels of one row."""
import numpy as np
import pytest

import oracle as O
import paper_1705_01387_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("R", [1, 3, 4, 5, 67, 1030])
@pytest.mark.parametrize("M", [1, 15, 16, 17, 64, 65, 130])
def test_kpm_of_many_rows(gpu, R, M):
    import torch
    print(f"case: kpm R={R} M={M}", flush=True)
    rng = np.random.default_rng(1000 * R + M)
    dE = 4.5
    for nE in (1, 2, 15, 16, 17, 65, 257, 300):
        C, g = rng.standard_normal((R, M)), rng.standard_normal((R, nE))
        E = rng.permutation(rng.uniform(-1, 1, nE)) * dE * (1 - 1e-6)
        for jackson in (True, False):
            basis = O.kpm_reconstruct(np.eye(M), E, dE, 10.0, damping=None if jackson else np.ones(M))   # [nE, M]
            got = P.gpuqt_kpm_reconstruct(torch.from_numpy(C).cuda(), E, dE, 10.0, jackson=jackson).cpu().numpy()
            want = C @ basis.T
            assert np.max(np.abs(got - want)) < 1e-10 * np.max(np.abs(want)), nE
            got = P.gpuqt_kpm_reconstruct_adjoint(torch.from_numpy(g).cuda(), E, M, dE, 10.0, jackson=jackson).cpu().numpy()
            want = g @ basis
            assert np.max(np.abs(got - want)) < 1e-10 * np.max(np.abs(want)), nE


def test_energies_outside_the_band(gpu):
    """NaN there and nowhere else; their weights add nothing to the transpose."""
    import torch
    print("case: kpm energies outside the band", flush=True)
    rng = np.random.default_rng(1)
    E = np.linspace(-5.0, 5.0, 300)
    for R in (2, 600):
        C, g = rng.standard_normal((R, 40)), rng.standard_normal((R, 300))
        out = P.gpuqt_kpm_reconstruct(torch.from_numpy(C).cuda(), E, 4.5, 10.0).cpu().numpy()
        assert np.array_equal(np.isnan(out), np.broadcast_to(np.abs(E) >= 4.5, out.shape))
        full = P.gpuqt_kpm_reconstruct_adjoint(torch.from_numpy(g).cuda(), E, 40, 4.5, 10.0).cpu().numpy()
        k = np.abs(E) < 4.5
        part = P.gpuqt_kpm_reconstruct_adjoint(torch.from_numpy(g[:, k]).cuda(), E[k], 40, 4.5, 10.0).cpu().numpy()
        assert np.max(np.abs(full - part)) < 1e-12 * np.max(np.abs(part))


def test_time_grows_with_the_work(gpu):
    """4096 rows: 256 energies of 32 moments, and one energy's 1000 moments back (a wavefront per energy took 610
    us, a workgroup per 8 moments 2,100; the work is 34 and 4 million terms, 10 and 26 us measured)."""
    import torch
    print("case: kpm times", flush=True)
    C, g = torch.randn(4096, 32, dtype=torch.float64, device="cuda"), torch.randn(4096, 1, dtype=torch.float64, device="cuda")
    E = np.linspace(-4.0, 4.0, 256)

    def best(call):
        call()
        t = []
        for _ in range(5):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            call()
            b.record()
            b.synchronize()
            t.append(1e3 * a.elapsed_time(b))
        return min(t)

    assert best(lambda: P.gpuqt_kpm_reconstruct(C, E, 4.5, 10.0)) < 250.0
    assert best(lambda: P.gpuqt_kpm_reconstruct_adjoint(g, np.array([0.3]), 1000, 4.5, 10.0)) < 500.0
