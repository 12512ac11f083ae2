"""Which calls go to the marches and patches, seen from the launches that gpuqt_timing counts (a march takes several
steps a launch, the general kernels one), and the marches' results on boxes large enough for them."""
import numpy as np
import pytest

import paper_1705_01387_amd as P
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-10
MARCH = 3 << 26


def vectors(n, B, seed):
    import torch
    return torch.from_numpy(I.random_phase(n, B, seed)).cuda()


def launches(H, family, call):
    """Steps per launch are more than one where a march ran: the launches of one call."""
    P.gpuqt_set_timing(H, True)
    P.gpuqt_timing(H)
    call()
    n = P.gpuqt_timing(H)[family][1]
    P.gpuqt_set_timing(H, False)
    return n


def marched(H, d, K):
    """Families that march K steps: moments of phi, evolution without and with the commutator, VAC rows."""
    return dict(sym=launches(H, "moment_sym", lambda: P.gpuqt_moments(H, d, d, 2 * K)) < K,
                evo=launches(H, "evolve", lambda: P.gpuqt_evolve(H, d, 0.1, K + 1)) < K,
                msd=launches(H, "msd", lambda: P.gpuqt_evolve(H, d, 0.1, K + 1, with_commutator=True)) < K,
                pair=launches(H, "moment_pair", lambda: P.gpuqt_vac(H, d, [0.1], 2 * K)) < K)


# Lattices whose general kernels are faster in every family, by 1.2 to 20 times, B = 1 and 4: boxes that
# do not fill the chip and strips whose tiles own a few of their cells.
GENERAL = {
    "box5": (lambda: I.cubic(5, W=2.0, seed=1), 1),
    "box20": (lambda: I.cubic(20, W=2.0, seed=1), 4),
    "box27": (lambda: I.cubic(27, W=2.0, seed=1), 1),
    "box_flat": (lambda: I.box(100, 100, 3, W=2.0, seed=1), 1),
    "box_thin": (lambda: I.box(3, 3, 3000, W=2.0, seed=1), 4),
    "box_strip": (lambda: I.box(5, 5, 4000, W=2.0, seed=1), 16),
    "strip_bonds": (lambda: I.bond_disorder(I.square(4, 22500, W=2.0, seed=1), 0.2, 2), 4),
    "strip_flux": (lambda: I.honeycomb(2, 22500, flux=1 / 45000, W=2.0, seed=1), 4),
}


@pytest.mark.parametrize("name", list(GENERAL))
def test_general_kernels_where_faster(gpu, name):
    print(f"case: route {name}", flush=True)
    make, B = GENERAL[name]
    m = make()
    H = P.gpuqt_build_h_from_model(m)
    assert H.info.kernel_variant & MARCH
    assert not any(marched(H, vectors(m.n, B, 3), 48).values())


def test_few_steps(gpu):
    """A single step of a launch of eight (the general kernels' too), and a series of one term, which has no step."""
    print("case: route of few steps", flush=True)
    m = I.square(1000, 900, W=2.0, seed=4)
    H = P.gpuqt_build_h_from_model(m)
    for B in (1, 2):
        d = vectors(m.n, B, 5)
        assert all(marched(H, d, 48).values())
        assert launches(H, "moment_sym", lambda: P.gpuqt_moments(H, d, d, 3)) == 1
        P.gpuqt_set_variant(H, H.info.kernel_variant & ~MARCH)
        ref = [P.gpuqt_moments(H, d, d, 3), P.gpuqt_evolve(H, d, 0.3, 1)]
        P.gpuqt_set_variant(H, MARCH)
        assert ((P.gpuqt_moments(H, d, d, 3) - ref[0]).abs().max() / ref[0].abs().max()).item() < TOL
        assert (P.gpuqt_evolve(H, d, 0.3, 1) - ref[1]).abs().max().item() < TOL


# Hermitian and evolution tiles of a box own 26 x 26 cells at most, the commutator's and the two chains' 28 x 28;
# runs of one plane and of several.
BOXES = {
    "26x53x44": (lambda: I.box(26, 53, 44, W=3.0, seed=6), 16),
    "28x57x40_shuffled": (lambda: I.box(28, 57, 40, W=3.0, seed=7, slot_seed=8), 16),
    "57x53x21": (lambda: I.box(57, 53, 21, W=3.0, seed=9), 16),
    "90x11x40": (lambda: I.box(90, 11, 40, W=3.0, seed=10), 16),
    "79x66x61": (lambda: I.box(79, 66, 61, W=3.0, seed=15), 4),
    "105x99x98": (lambda: I.box(105, 99, 98, W=3.0, seed=16), 1),
}


def against_general(H, call):
    """{name: tensor} of call with the marches and without."""
    code = H.info.kernel_variant
    on = call()
    P.gpuqt_set_variant(H, code & ~MARCH)
    off = call()
    P.gpuqt_set_variant(H, code)
    for k, ref in off.items():
        assert ((on[k] - ref).abs().max() / ref.abs().max()).item() < TOL, k


@pytest.mark.parametrize("name", list(BOXES))
def test_box_marches(gpu, name):
    """Boxes that march every family but the two chains, against the general kernels."""
    print(f"case: box march {name}", flush=True)
    make, B = BOXES[name]
    m = make()
    H = P.gpuqt_build_h_from_model(m)
    d, c = vectors(m.n, B, 11), vectors(m.n, B, 12)
    on = marched(H, d, 48)
    assert on["sym"] and on["evo"] and on["msd"], on
    against_general(H, lambda: dict(
        mu=P.gpuqt_moments(H, d, d, 50), odd=P.gpuqt_moments(H, d, d, 63), one=P.gpuqt_evolve(H, d, -1.9),
        chi=P.gpuqt_evolve(H, d, 1.9, chi=c, with_commutator=True)[1],
        zero=P.gpuqt_evolve(H, d, 1.9, with_commutator=True)[1], msd=P.gpuqt_msd(H, d, [1.0, 1.3], 40)))


@pytest.mark.parametrize("name", list(BOXES))
def test_box_vac_marches(gpu, name):
    """A VAC series of few moments and long steps: there the marches of the two-vector evolution outweigh those of the
    two chains, and both run; recorded rows and their tape's gradients as well."""
    import torch
    print(f"case: box VAC march {name}", flush=True)
    make, B = BOXES[name]
    m = make()
    H = P.gpuqt_build_h_from_model(m)
    d, dts, M = vectors(m.n, B, 13), [4.0, 0.5, 3.0], 11
    assert launches(H, "moment_pair", lambda: P.gpuqt_vac(H, d, dts, M)) < 3 * (M // 2)
    w = torch.from_numpy(np.random.default_rng(14).normal(size=(3, 1, B, M))).cuda()

    def rows():
        out, tape = P.gpuqt_vac_record(H, d, dts, M)
        assert torch.equal(out, P.gpuqt_vac(H, d, dts, M))
        return dict(rows=out, tape=P.gpuqt_vac_backward_tape(H, d, dts, w, tape)[0])

    against_general(H, rows)
