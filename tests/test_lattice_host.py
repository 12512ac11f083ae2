"""CPU tests of the lattice recognition that chooses the march and patch kernels: whatever a recognised
pattern says about neighbours and hoppings has to be the matrix of the descriptor, row by row and bit for bit
(lattice_host.cpp compares it with the layout that the general kernels read)."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

from paper_1705_01387_amd import inputs as I

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_1705_01387_amd", "csrc")
NONE, SQUARE, BRICK, BOX, CHAIN, NNN = range(6)


@pytest.fixture(scope="module")
def lat(tmp_path_factory):
    cxx, rocm = shutil.which("g++"), os.environ.get("ROCM_PATH", "/opt/rocm")
    if cxx is None or not os.path.isdir(os.path.join(rocm, "include", "hip")):
        pytest.skip("no host compiler or no HIP headers")
    so = str(tmp_path_factory.mktemp("lattice") / "lattice_host.so")
    subprocess.check_call([cxx, "-O1", "-std=c++17", "-D__HIP_PLATFORM_AMD__", "-I", os.path.join(rocm, "include"), "-shared",
                           "-fPIC", os.path.join(HERE, "lattice_host.cpp"), os.path.join(CSRC, "lattice.cpp"),
                           os.path.join(CSRC, "layout.cpp"), "-o", so])
    return ctypes.CDLL(so)


def check(lat, nn, nbr, hop, x=None, length_x=0.0, seg_offsets=None, no_dictionary=False, check_hermitian=False):
    """lattice_check: the pattern, + 100 where it is not the descriptor's matrix, -1 refused."""
    nn, nbr = np.ascontiguousarray(nn, np.int32), np.ascontiguousarray(nbr, np.int32)
    n = nn.shape[0]
    cplx = hop is not None and np.iscomplexobj(hop)
    hop = None if hop is None else np.ascontiguousarray(hop, np.complex128 if cplx else np.float64)
    x = np.zeros(n) if x is None else np.ascontiguousarray(x, np.float64)
    off = None if seg_offsets is None else np.ascontiguousarray(seg_offsets, np.int64)
    p = lambda a: None if a is None else a.ctypes.data_as(ctypes.c_void_p)
    return lat.lattice_check(ctypes.c_int64(n), nbr.shape[1], p(nn), p(nbr), p(hop), int(cplx), p(x),
                             ctypes.c_double(length_x), 1 if off is None else len(off) - 1, p(off), int(no_dictionary),
                             int(check_hermitian), None)


def model(lat, m, **kw):
    return check(lat, m.nn, m.nbr, m.hop, m.x, m.length_x, **kw)


def permuted(m, seed):
    """The same order of neighbours on every row, another one than the natural."""
    order = np.random.default_rng(seed).permutation(m.nbr.shape[1])
    m.nbr = m.nbr[:, order]
    m.hop = None if m.hop is None else m.hop[:, order]
    return m


MODELS = {
    "square": (SQUARE, lambda: I.square(9, 7, seed=1)),
    "square3x3": (SQUARE, lambda: I.square(3, 3, seed=1, t1=-0.4)),
    "square_bonds": (SQUARE, lambda: permuted(I.bond_disorder(I.square(8, 5), 0.2, 2, max_phase=0.4), 3)),
    "open": (SQUARE, lambda: I.square(6, 7, periodic_x=False)),
    "brick": (BRICK, lambda: I.honeycomb(4, 6)),
    "brick_flux": (BRICK, lambda: permuted(I.honeycomb(5, 8, flux=1 / 40), 4)),
    "brick_bonds": (BRICK, lambda: permuted(I.bond_disorder(I.honeycomb(6, 10), 0.3, 5), 6)),
    "box": (BOX, lambda: I.box(5, 4, 3, slot_seed=7)),
    "chain3": (CHAIN, lambda: I.chain(3)),
    "chain_bonds": (CHAIN, lambda: permuted(I.bond_disorder(I.chain(70), 0.2, 8, max_phase=0.3), 9)),
    "nnn": (NNN, lambda: I.square(5, 6, t2=-0.2)),
    "nnn3x3": (NNN, lambda: permuted(I.square(3, 3, t2=-0.2), 10)),
    "nnn_uniform": (NNN, lambda: permuted(I.square(4, 9, t1=-0.5, t2=-0.5), 11)),
    "nnn_bonds": (NNN, lambda: permuted(I.bond_disorder(I.square(7, 4, t2=-0.3), 0.2, 12, max_phase=0.3), 13)),
}


@pytest.mark.parametrize("no_dictionary", [False, True])
@pytest.mark.parametrize("name", list(MODELS))
def test_recognised_pattern_is_the_matrix(lat, name, no_dictionary):
    want, make = MODELS[name]
    assert model(lat, make(), no_dictionary=no_dictionary, check_hermitian=True) == want


def test_repeated_neighbour_in_the_first_row(lat):
    """Row 0 of a square with next-nearest neighbours names -x twice, half the hopping each, and +x not at all
    (Hermitian: the entry back is 0): legal, duplicates are summed, and not the pattern's matrix."""
    m = I.square(5, 6, t2=-0.2)
    hop = m.hop.copy()
    xp, xm = [int(np.flatnonzero(m.nbr[0] == c)[0]) for c in (1, 4)]
    back = int(np.flatnonzero(m.nbr[1] == 0)[0])
    m.nbr[0, xp] = m.nbr[0, xm]
    hop[0, xp] = hop[0, xm] = 0.5 * hop[0, xm]
    hop[1, back] = 0.0
    for no_dictionary in (False, True):
        assert check(lat, m.nn, m.nbr, hop, no_dictionary=no_dictionary, check_hermitian=True) == NONE


@pytest.mark.parametrize("name", ["square_bonds", "brick_flux", "brick_bonds", "chain_bonds", "nnn", "nnn3x3", "nnn_uniform",
                                  "nnn_bonds", "square", "open", "box"])
def test_altered_neighbours_are_refused(lat, name):
    """One entry of one row pointing elsewhere (another neighbour of the row, so that one is named twice, or any
    site), for the first rows, row Lx and the last one, and all rows alike: never another matrix's pattern."""
    want, make = MODELS[name]
    rng = np.random.default_rng(14)
    for row in (0, 0, 0, 1, 2, "last", "all"):
        for j in range(make().nbr.shape[1]):
            m = make()
            rows = slice(None) if row == "all" else m.n - 1 if row == "last" else row
            i = 0 if row == "all" else rows
            if j >= m.nn[i]:
                continue
            k = int(rng.integers(0, m.nn[i] - 1))
            k += k >= j
            if row == "all" or rng.random() < 0.7:
                m.nbr[rows, j] = m.nbr[rows, k]
            else:
                m.nbr[rows, j] = int(rng.integers(0, m.n))
            for no_dictionary in (False, True):
                assert model(lat, m, no_dictionary=no_dictionary) < 100, (row, j)


def test_segments_and_row_orders(lat):
    """Segments are recognised together only where their neighbours are stored in the same order; with one
    order per row only one hopping will do."""
    mods = [I.square(5, 6, t2=-0.2), I.square(4, 3, t2=-0.2)]
    cat = I.concat_segments(mods)
    off = np.cumsum([0] + [m.n for m in mods])
    assert check(lat, cat.nn, cat.nbr, cat.hop, seg_offsets=off) == NNN
    nbr, hop = cat.nbr.copy(), cat.hop.copy()
    nbr[30:, [0, 1]], hop[30:, [0, 1]] = nbr[30:, [1, 0]], hop[30:, [1, 0]]
    assert check(lat, cat.nn, nbr, hop, seg_offsets=off) == NONE
    m = I.bond_disorder(I.square(6, 5), 0.2, 15)
    order = np.argsort(np.random.default_rng(16).random(m.nbr.shape), axis=1)
    nbr = np.take_along_axis(m.nbr, order, 1)
    assert check(lat, m.nn, nbr, np.take_along_axis(m.hop, order, 1), no_dictionary=True) == NONE
    assert check(lat, m.nn, nbr, None) == SQUARE
