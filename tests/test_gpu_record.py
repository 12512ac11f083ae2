"""gpuqt_vac_record on lattices with marches, whose tape holds rows of B columns while the marches' own vectors
are planar: its rows are gpuqt_vac's bit for bit, with any number of terms a step, and the gradients from its
tape are those of gpuqt_vac_backward, which records nothing.  Bar: normwise 1e-10."""
import numpy as np
import pytest

import paper_1705_01387_amd as P
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-10
MARCH = 3 << 26


def err(got, ref):
    return float((got - ref).abs().max() / ref.abs().max().clamp(min=1e-300))


def vectors(n, B, seed):
    import torch
    return torch.from_numpy(I.random_phase(n, B, seed)).cuda()


def segments(mods, **kw):
    """One handle of several models, each with the DeltaE of its own disorder."""
    cat = I.concat_segments(mods)
    return P.gpuqt_build_h(cat.nn, cat.nbr, cat.hop, cat.onsite, cat.x, 0.0, cat.volume, 0.0,
                           seg_offsets=np.cumsum([0] + [m.n for m in mods]), seg_length_x=[m.length_x for m in mods], **kw)


SETS = {
    "squares": lambda: segments([I.square(20, 12, W=6.0, seed=1), I.square(9, 31, W=0.5, seed=2)]),
    "bricks": lambda: segments([I.honeycomb(8, 10, W=8.0, seed=3), I.honeycomb(5, 8, W=0.5, seed=4)]),
    "chains": lambda: segments([I.chain(300, W=5.0, seed=5), I.chain(77, W=0.3, seed=6)]),
    "nnn": lambda: segments([I.square(13, 9, W=6.0, seed=7, t2=-0.2), I.square(8, 8, W=0.5, seed=8, t2=-0.2)]),
}


@pytest.mark.parametrize("Np", [1, 2, 3, 7])
@pytest.mark.parametrize("B", [1, 2, 4])
@pytest.mark.parametrize("name", list(SETS))
def test_record_of_segments_with_few_terms(gpu, name, B, Np):
    """Segments of different DeltaE, so that J_m(DeltaE dt) differs between their rows."""
    import torch
    print(f"case: record {name} B={B} Np={Np}", flush=True)
    H = SETS[name]()
    assert H.energy_max[0] > 1.3 * H.energy_max[1] and H.info.kernel_variant & MARCH == MARCH
    d, dts, M = vectors(H.n, B, 10), [0.4, 0.9, 0.2], 13
    w = torch.from_numpy(np.random.default_rng(11).normal(size=(3, 2, B, M))).cuda()
    rows, tape = P.gpuqt_vac_record(H, d, dts, M, Np)
    assert torch.equal(rows, P.gpuqt_vac(H, d, dts, M, Np))
    taped = P.gpuqt_vac_backward_tape(H, d, dts, w, tape, Np=Np)[0]
    P.gpuqt_set_variant(H, 0)
    assert err(rows, P.gpuqt_vac(H, d, dts, M, Np)) < TOL
    assert err(taped, P.gpuqt_vac_backward(H, d, dts, w, Np=Np)[0]) < TOL
