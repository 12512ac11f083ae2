"""The reconstruction and its transpose at counts of moments and energies around the sizes their kernels
work in: 64 lanes and tiles of 1024 moments, 8 energies or 8 moments a workgroup.  Bar: normwise
1e-10; T_n(x) = cos(n acos x) is off by at most a few n ulps either way (1e-12 at 4,000 moments)."""
import numpy as np
import pytest

import oracle as O
import paper_1705_01387_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M", [1, 2, 7, 63, 64, 65, 1023, 1024, 1025, 2500])
@pytest.mark.parametrize("nE", [1, 7, 8, 9, 257])
def test_kpm_and_transpose(gpu, M, nE):
    import torch
    print(f"case: kpm M={M} nE={nE}", flush=True)
    rng = np.random.default_rng(1000 * nE + M)
    C, dE = rng.standard_normal((3, M)), 4.5
    E = np.sort(rng.uniform(-1, 1, nE)) * dE * (1 - 1e-6)
    for jackson in (True, False):
        damp = None if jackson else np.ones(M)
        got = P.gpuqt_kpm_reconstruct(torch.from_numpy(C).cuda(), E, dE, 10.0, jackson=jackson).cpu().numpy()
        ref = O.kpm_reconstruct(C.T, E, dE, 10.0, damping=damp).T
        assert np.max(np.abs(got - ref)) < 1e-10 * np.max(np.abs(ref))
        g = rng.standard_normal((3, nE))
        back = P.gpuqt_kpm_reconstruct_adjoint(torch.from_numpy(g).cuda(), E, M, dE, 10.0, jackson=jackson).cpu().numpy()
        basis = O.kpm_reconstruct(np.eye(M), E, dE, 10.0, damping=damp)      # [nE, M]
        want = g @ basis
        assert np.max(np.abs(back - want)) < 1e-10 * np.max(np.abs(want))
    out = P.gpuqt_kpm_reconstruct(torch.from_numpy(C).cuda(), np.array([dE, -dE, 5.0, 0.3]), dE, 10.0).cpu().numpy()
    assert np.isnan(out[:, :3]).all() and np.isfinite(out[:, 3]).all()
