"""Class gradients at every row width that the reverse steps are built for (3, 4, 6 and 8 neighbours, other and ragged widths),
with classes by bond (terms from the transposed product) and by direction (terms of the forward product), alone and
together with per-entry gradients, against the oracle.  With every vector kept, directed classes share a bond's terms out
differently: there the classes' sum is compared.  Bar: normwise 1e-10."""
import numpy as np
import pytest

import oracle as O
import paper_1705_01387_amd as P
from oracle.adjoint import class_parts
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-10
LATTICES = {
    "chain": lambda: I.bond_disorder(I.chain(90, W=1.0, seed=1), 0.2, 2, max_phase=0.3),
    "honeycomb": lambda: I.bond_disorder(I.honeycomb(7, 8, W=1.0, seed=3), 0.2, 4, max_phase=0.3),
    "square": lambda: I.bond_disorder(I.square(11, 9, W=1.0, seed=5), 0.2, 6),
    "box": lambda: I.bond_disorder(I.box(5, 4, 6, W=1.0, seed=7), 0.2, 8, max_phase=0.3),
    "nnn": lambda: I.bond_disorder(I.square(9, 10, W=1.0, seed=9, t2=-0.3), 0.2, 10),
    "open": lambda: I.bond_disorder(I.square(10, 9, W=1.0, seed=11, periodic_x=False), 0.2, 12),
}


@pytest.mark.parametrize("storage", [{}, dict(no_dictionary=True)])
@pytest.mark.parametrize("n_class", [1, 2, 4])
@pytest.mark.parametrize("directed", [True, False])
@pytest.mark.parametrize("name", list(LATTICES))
def test_class_gradients(gpu, name, directed, n_class, storage):
    import torch
    print(f"case: reverse widths {name} directed={directed} classes={n_class} {storage}", flush=True)
    m = LATTICES[name]()
    lo, hi = np.minimum(np.arange(m.n)[:, None], m.nbr), np.maximum(np.arange(m.n)[:, None], m.nbr)
    m.hop_class = (np.random.default_rng(13).integers(0, n_class, m.nbr.shape) if directed else (lo * 7 + hi * 3) % n_class)
    m.hop_class = np.where(np.arange(m.nbr.shape[1]) < m.nn[:, None], m.hop_class, 0).astype(np.int32)
    m.n_class = n_class
    Hs, _, _ = O.operators(m.nn, m.nbr, m.hop, m.onsite, m.x, m.length_x)
    dE = 1.01 * O.gershgorin_bound(Hs)
    H = P.gpuqt_build_h_from_model(m, energy_max=dE, **storage)
    parts = class_parts(m.nn, m.nbr, m.hop, m.hop_class, n_class)
    zeros = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")
    err = lambda got, ref: np.max(np.abs(got.cpu().numpy() - ref)) / np.max(np.abs(ref))
    for B in (1, 2):
        L, R = I.random_phase(m.n, B, 14), I.random_phase(m.n, B, 15)
        dL, dR = torch.from_numpy(L).cuda(), torch.from_numpy(R).cuda()
        w = np.random.default_rng(16).normal(size=(1, B, 21))
        dw = torch.from_numpy(w).cuda()
        for a, b, da, db in ((L, R, dL, dR), (L, L, dL, dL)):
            rU, rC = O.moments_gradient(Hs, a, b, dE, w[0].T, parts)
            for stride in (0, 1):
                entry = None
                for both in (False, True):
                    gH = zeros(m.n, int(H.info.max_nn), 2) if both else None
                    gU, gC = P.gpuqt_moments_backward(H, da, db, dw, None, zeros(n_class), ckpt_stride=stride, grad_hop=gH)[:2]
                    assert err(gU, rU) < TOL, (B, stride, both)
                    if directed and stride == 1 and not both:
                        assert abs(gC.sum().item() - rC.sum()) < TOL * np.max(np.abs(rC)), (B, stride)
                    else:
                        assert err(gC, rC) < TOL, (B, stride, both)
                    if both:      # the same per-entry gradients as without class sums
                        alone = zeros(*gH.shape)
                        P.gpuqt_moments_backward(H, da, db, dw, None, None, ckpt_stride=stride, grad_hop=alone)
                        assert ((gH - alone).abs().max() / alone.abs().max()).item() < TOL
