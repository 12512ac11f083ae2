"""Rows wider than gpuqt_build_h looks at for Hermitian classes (128 entries): class gradients against the oracle on both
sides of that width, and a handle of wide rows built in the time of one whose classes it never looks at."""
import time

import numpy as np
import pytest

import oracle as O
import paper_1705_01387_amd as P
from oracle.adjoint import class_parts
from paper_1705_01387_amd import inputs as I

pytestmark = pytest.mark.gpu
TOL = 1e-10


def circulant(n, width, seed):
    """Rows with the same random offsets, paired with their opposites."""
    o = np.sort(np.random.default_rng(seed).choice(np.arange(1, n // 2), width // 2, replace=False))
    o = np.concatenate([o, n - o])
    return ((np.arange(n)[:, None] + o[None]) % n).astype(np.int32)


@pytest.mark.parametrize("width", [126, 128, 130, 200])
def test_class_gradients_of_wide_rows(gpu, width):
    import torch
    print(f"case: class gradients of rows of {width}", flush=True)
    n, C = 420, 3
    nbr = circulant(n, width, 1)
    nn = np.full(n, width, np.int32)
    lo, hi = np.minimum(np.arange(n)[:, None], nbr), np.maximum(np.arange(n)[:, None], nbr)
    cls = ((lo * 7 + hi * 3) % C).astype(np.int32)
    hop = -1.0 - 0.1 * ((lo * 5 + hi * 11) % 13)
    on, x = I.anderson(n, 1.0, 2), np.zeros(n)
    Hs, _, _ = O.operators(nn, nbr, hop, on, x, 0.0)
    dE = 1.01 * O.gershgorin_bound(Hs)
    H = P.gpuqt_build_h(nn, nbr, hop, on, x, 0.0, 1.0, dE, hop_class=cls, n_class=C)
    L, R = I.random_phase(n, 2, 3), I.random_phase(n, 2, 4)
    w = np.random.default_rng(5).normal(size=(1, 2, 30))
    parts = class_parts(nn, nbr, hop, cls, C)
    for stride in (0, 1):
        for a, b in ((L, R), (L, L)):
            da = torch.from_numpy(a).cuda()
            db = da if a is b else torch.from_numpy(b).cuda()
            gU, gC = P.gpuqt_moments_backward(H, da, db, torch.from_numpy(w).cuda(), None,
                                              torch.zeros(C, dtype=torch.float64, device="cuda"), ckpt_stride=stride)[:2]
            rU, rC = O.moments_gradient(Hs, a, b, dE, w[0].T, parts)
            assert np.max(np.abs(gU.cpu().numpy() - rU)) < TOL * np.max(np.abs(rU))
            assert np.max(np.abs(gC.cpu().numpy() - rC)) < TOL * np.max(np.abs(rC))


def test_build_time_of_wide_rows(gpu):
    """Five classes have no class gradients, so nothing is looked at: 33 ms; with one class the look took 430 more."""
    import torch
    print("case: build time of wide rows", flush=True)
    n, width = 4096, 1024
    nbr = circulant(n, width, 6)
    nn, cls = np.full(n, width, np.int32), np.zeros((n, width), np.int32)

    def best(**kw):
        t = []
        for _ in range(3):
            torch.cuda.synchronize()
            a = time.perf_counter()
            P.gpuqt_build_h(nn, nbr, None, np.zeros(n), np.zeros(n), 0.0, 1.0, **kw)
            torch.cuda.synchronize()
            t.append(time.perf_counter() - a)
        return min(t)

    assert best() < 5.0 * best(hop_class=cls, n_class=5)
