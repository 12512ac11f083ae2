"""The marches that store every step in rows of B columns (the forward vectors of the gradients and the chains of a recorded
VAC), on lattices too large for patches: gradients and recorded rows against the general kernels on the same
handle (variant bit 26 off), the recorded rows bit for bit against gpuqt_vac.  Bar: normwise 1e-10."""
import numpy as np
import pytest

import paper_1705_01387_amd as P
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-10
MARCH = 3 << 26


def sheet(Lx, Ly, seed, **kw):
    return I.square(Lx, Ly, W=2.0, seed=seed, **kw)


def segments(mods):
    cat = I.concat_segments(mods)
    return P.gpuqt_build_h(cat.nn, cat.nbr, cat.hop, cat.onsite, cat.x, 0.0, cat.volume, 0.0,
                           seg_offsets=np.cumsum([0] + [m.n for m in mods]), seg_length_x=[m.length_x for m in mods])


def one(m, **kw):
    return P.gpuqt_build_h_from_model(m, **kw)


# widths at and one past a tile's 48 or 112 (T = 8), 54 (T = 5), 56 (T = 4), 58 (T = 3) owned cells; B: marches, not patches
CASES = {
    "square": (lambda: one(sheet(48 * 12 + 1, 203, 1)), 16),
    "square_narrow": (lambda: one(sheet(54 * 2, 2000, 2)), 4),
    "square_bonds": (lambda: one(I.bond_disorder(sheet(56 * 7, 303, 3), 0.2, 4, max_phase=0.5), no_dictionary=True), 16),
    "square_real_bonds": (lambda: one(I.bond_disorder(sheet(400, 301, 5), 0.2, 6), no_dictionary=True, slice_height=32), 4),
    "open": (lambda: one(sheet(48 * 9 + 2, 277, 7, periodic_x=False)), 16),
    "brick_flux": (lambda: one(I.honeycomb(125, 486, flux=1 / (125 * 486), W=2.0, seed=8)), 16),
    "brick_bonds": (lambda: one(I.honeycomb(130, 440, flux=1 / 57200, W=2.0, seed=9), no_dictionary=True), 4),
    "segments": (lambda: segments([sheet(300, 211, 10), sheet(117, 400, 11), sheet(49, 50, 12)]), 8),
    "box": (lambda: one(I.box(26, 53, 44, W=3.0, seed=13)), 16),
    "patches": (lambda: one(sheet(190, 121, 14, t2=-0.2)), 4),
}


def vectors(n, B, seed):
    import torch
    return torch.from_numpy(I.random_phase(n, B, seed)).cuda()


@pytest.mark.parametrize("name", list(CASES))
def test_kept_steps(gpu, name):
    import torch
    print(f"case: kept steps {name}", flush=True)
    make, B = CASES[name]
    H = make()
    n, S, K = H.n, H.n_segments, int(H.info.max_nn)
    code = H.info.kernel_variant
    assert code & MARCH == MARCH
    L, R = vectors(n, B, 20), vectors(n, B, 21)
    rng = np.random.default_rng(22)
    zeros = lambda *s: torch.zeros(s, dtype=torch.float64, device="cuda")
    dts = [0.7, 0.4]
    ran = {}

    def outputs(tag):
        out = {}
        for M in (49, 20):
            P.gpuqt_set_timing(H, True)
            w = torch.from_numpy(rng_w[M]).cuda()
            for kind, a, b in (("sym", L, L), ("pair", L, R)):
                gU, gC = P.gpuqt_moments_backward(H, a, b, w, zeros(n), zeros(int(H.info.n_class)), ckpt_stride=1)[:2]
                out[f"{kind}{M}_U"], out[f"{kind}{M}_C"] = gU, gC
            P.gpuqt_set_timing(H, False)
            gU, gH = zeros(n), zeros(n, K, 2)
            P.gpuqt_moments_backward(H, L, R, w, gU, grad_hop=gH, ckpt_stride=1)
            out[f"entry{M}_U"], out[f"entry{M}_H"] = gU, gH
        ran[tag] = {f: c for f, (_, c) in P.gpuqt_timing(H).items()}
        w = torch.from_numpy(rng_w["vac"]).cuda()
        rows, tape = P.gpuqt_vac_record(H, L, dts, 21)
        assert torch.equal(rows, P.gpuqt_vac(H, L, dts, 21))
        out["rows"] = rows
        out["tape_U"], out["tape_C"] = P.gpuqt_vac_backward_tape(H, L, dts, w, tape, zeros(n), zeros(int(H.info.n_class)))
        return out

    rng_w = {M: rng.normal(size=(S, B, M)) for M in (49, 20)}
    rng_w["vac"] = rng.normal(size=(2, S, B, 21))
    on = outputs("march")
    P.gpuqt_set_variant(H, code & ~MARCH)
    off = outputs("general")
    for k, ref in off.items():
        assert ((on[k] - ref).abs().max() / ref.abs().max()).item() < TOL, k
    steps = 24 + 10
    assert ran["general"]["moment_sym"] == steps and ran["general"]["moment_pair"] == steps
    assert ran["march"]["moment_sym"] < steps
    assert name == "box" or ran["march"]["moment_pair"] < steps
