"""Class gradients where a bond's two directions are in different classes (the class's hoppings are not
Hermitian by themselves), so that the terms cannot be taken from the transposed product: against the oracle's
reverse recurrence.  With every vector kept (stride 1) the moments come from products <a_k|b_k>, which share out a
bond's terms between its directions' classes differently: there the classes' sum is compared.  Bar:
normwise 1e-10."""
import numpy as np
import pytest

import oracle as O
import paper_1705_01387_amd as P
from oracle.adjoint import class_parts, vac_gradient, velocity_class_parts
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-10


def err(got, ref):
    return float(np.max(np.abs(got.cpu().numpy() - ref)) / max(np.max(np.abs(ref)), 1e-300))


@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("storage", [{}, dict(no_dictionary=True)])
@pytest.mark.parametrize("stride", [0, 1, 7])
@pytest.mark.parametrize("n_class", [2, 3])
def test_directed_classes(gpu, directed, storage, stride, n_class):
    import torch
    print(f"case: class gradients directed={directed} {storage} stride={stride} classes={n_class}", flush=True)
    m = I.honeycomb(9, 10, flux=1 / 90, W=1.0, seed=1)
    if directed:
        m.hop_class = np.random.default_rng(2).integers(0, n_class, m.nbr.shape).astype(np.int32)
    else:      # by bond
        lo, hi = np.minimum(np.arange(m.n)[:, None], m.nbr), np.maximum(np.arange(m.n)[:, None], m.nbr)
        m.hop_class = ((lo * 7 + hi * 3) % n_class).astype(np.int32)
    m.n_class = n_class
    Hs, V, _ = O.operators(m.nn, m.nbr, m.hop, m.onsite, m.x, m.length_x)
    dE = 1.01 * O.gershgorin_bound(Hs)
    H = P.gpuqt_build_h_from_model(m, energy_max=dE, **storage)
    parts = class_parts(m.nn, m.nbr, m.hop, m.hop_class, n_class)
    L, R = I.random_phase(m.n, 2, 3), I.random_phase(m.n, 2, 4)
    dL, dR = torch.from_numpy(L).cuda(), torch.from_numpy(R).cuda()
    w = np.random.default_rng(5).normal(size=(1, 2, 33))
    dw = torch.from_numpy(w).cuda()

    def same(got, ref, kept):
        if directed and kept:
            return abs(got.sum().item() - ref.sum()) < TOL * np.max(np.abs(ref))
        return err(got, ref) < TOL

    zero = lambda: torch.zeros(n_class, dtype=torch.float64, device="cuda")
    for a, b, da, db in ((L, R, dL, dR), (L, L, dL, dL)):
        gU, gC = P.gpuqt_moments_backward(H, da, db, dw, None, zero(), ckpt_stride=stride)[:2]
        rU, rC = O.moments_gradient(Hs, a, b, dE, w[0].T, parts)
        assert err(gU, rU) < TOL and same(gC, rC, stride == 1)
    dts = [0.4, 0.0, 1.1]
    w = np.random.default_rng(6).normal(size=(3, 1, 2, 20))
    gU, gC = P.gpuqt_vac_backward(H, dL, dts, torch.from_numpy(w).cuda(), ckpt_stride=min(stride, 1), grad_class=zero())
    Vc = velocity_class_parts(m.nn, m.nbr, m.hop, m.hop_class, n_class, m.x, m.length_x)
    rU, rC = vac_gradient(Hs, V, L, dts, dE, 20, np.transpose(w[:, 0], (0, 2, 1)), 0, parts, Vc)
    assert err(gU, rU) < TOL and same(gC, rC, stride > 0)
