"""Performance cases of the library: the calls its users make, over the sizes they make them at.

Every case names one operation on one lattice:

  dos     Chebyshev moments of a block of random-phase vectors and the KPM density of states
  vac     velocity-autocorrelation rows (gpuqt_vac)
  msd     mean-square-displacement rows (gpuqt_msd)
  evolve  one time step of wave packets (gpuqt_evolve), with or without the commutator series
  train   forward and backward of a loss on the density of states and the VAC rows (autograd)
  bonds   gradient of a moment loss for every stored hopping (gpuqt_moments_backward)

`lattice` is square, nnn (square with next-nearest neighbours in a second hopping class),
honeycomb (brick-wall form), cubic, chain or squares (segments of growing squares);
`hop` is uniform, flux (Peierls phases of a uniform field), table or entries (per-bond disorder,
complex).  `tune` says whether the program calls the autotuner on its handle, as a long
calculation does, or not, as the folder driver does.
"""
import functools
import math

import numpy as np
import torch

import paper_1705_01387_amd as P
from paper_1705_01387_amd import autograd as A

C128 = torch.complex128


def _case(name, op, lattice, dims, B=1, M=1000, W=2.0, hop="uniform", n_t=0, dt=0.0, Np=0, nE=0, tune=True,
          open_x=False, commutator=False):
    Lx, Ly, Lz = (tuple(dims) + (1, 1))[:3]
    c = dict(op=op, lattice=lattice, Lx=Lx, Ly=Ly, Lz=Lz, B=B, M=M, W=W, hop=hop, n_t=n_t, dt=dt, Np=Np, nE=nE,
             tune=tune, open_x=open_x, commutator=commutator)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # the smallest call: a 64 x 64 sample whose vectors are a few cache lines per compute unit
        _case("dos_square64", "dos", "square", (64, 64), M=1000, W=1.0, nE=1001),
        # the folder driver's path: no tuning, open boundary, a ragged size, a pair of vectors
        _case("dos_square_open_b2", "dos", "square", (777, 613), B=2, M=500, nE=601, tune=False, open_x=True),
        # density of states of a disordered cubic sample with the default single random vector
        _case("dos_cubic_b1", "dos", "cubic", (160, 144, 121), M=1000, W=8.0, nE=801),
        # the benchmark's step: one MSD time step of a block of four on 8,000,000 orbitals
        _case("msd_cubic200_b4", "msd", "cubic", (200, 200, 200), B=4, M=1000, W=16.0, n_t=1, dt=2.0, Np=60),
        # disorder average: eight uneven realisations x 16 vectors in one call
        _case("dos_squares_b16", "dos", "squares", (200, 2000, 8), B=16, M=200, nE=201),
        # the method's two published examples: diffusive square and localized chain
        _case("vac_square2000", "vac", "square", (2000, 2000), M=1000, W=4.0, n_t=3, dt=0.2),
        _case("msd_chain4m_b2", "msd", "chain", (4_000_000,), B=2, M=500, W=4.0, n_t=2, dt=1.0),
        # graphene in a magnetic field: complex hoppings from a table, long time steps
        _case("vac_honeycomb2m", "vac", "honeycomb", (2000, 1000), M=1000, hop="flux", n_t=2, dt=22.789),
        # the same lattice with every bond its own complex number, a block of vectors
        _case("dos_honeycomb_bonds_b4", "dos", "honeycomb", (1000, 702), B=4, M=400, hop="entries", nE=401),
        # wave packets propagated on a real-space grid: outputs are the states themselves
        _case("evolve_square_b2", "evolve", "square", (1531, 1024), B=2, n_t=1, dt=10.0),
        # fitting a Hamiltonian: forward and backward of a spectral and transport loss
        _case("train_nnn512", "train", "nnn", (512, 512), M=512, W=2.0, hop="table", n_t=10, dt=1.0, nE=1001),
        # a gradient for every bond of a disordered sample
        _case("bonds_square256_b2", "bonds", "square", (256, 193), B=2, M=256, hop="entries"),
    ]


def draw(rng):
    def logint(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    op = rng.choice(["dos", "dos", "dos", "vac", "msd", "msd", "evolve", "train", "bonds"])
    lattice = {"train": "nnn", "bonds": rng.choice(["square", "honeycomb"])}.get(
        op, rng.choice(["square", "square", "honeycomb", "cubic", "chain", "squares", "nnn"]))
    n = logint(2_000, {"train": 260_000, "bonds": 60_000}.get(op, 4_000_000))
    B = 1 if op == "train" else rng.choice([1, 1, 2, 4, 8, 16])
    n_t = {"vac": rng.randint(1, 3), "msd": rng.randint(1, 3), "evolve": 1, "train": rng.randint(2, 5)}.get(op, 0)
    M = logint(48, 512 if op == "train" else 256 if op == "bonds" else 1200)
    dt = round(rng.uniform(0.2, 12.0), 3) if n_t else 0.0
    open_x = op in ("dos", "evolve") and lattice == "square" and rng.random() < 0.3
    hop = {"honeycomb": rng.choice(["uniform", "flux", "entries"]), "nnn": "table",
           "square": rng.choice(["uniform", "uniform", "entries"])}.get(lattice, "uniform")
    if op == "bonds":
        hop = "entries"
    if open_x:
        hop = "uniform"
    # the whole calculation costs no more than a third of the largest listed one
    steps = {"dos": M / 2, "vac": n_t * (M + 30 * dt), "msd": n_t * (M / 2 + 40 * dt), "evolve": 10 * dt}
    while n * B * steps.get(op, 0) > 6e9:
        n, B, M = (n, B // 2, M) if B > 1 else (n, B, M // 2) if M > 64 and op != "evolve" else (n // 2, B, M)
        steps = {"dos": M / 2, "vac": n_t * (M + 30 * dt), "msd": n_t * (M / 2 + 40 * dt), "evolve": 10 * dt}
    r = math.exp(rng.uniform(-0.8, 0.8))
    if lattice == "chain":
        dims = (n,)
    elif lattice == "cubic":
        a = n ** (1 / 3)
        s = math.exp(rng.uniform(-0.4, 0.4))
        dims = (max(5, round(a * s)), max(5, round(a / s * r ** 0.4)), max(5, round(a * r ** -0.4)))
    elif lattice == "squares":
        k = rng.randint(2, 8)
        hi = max(24, round(math.sqrt(2 * n / k)))
        dims = (max(8, hi // rng.randint(2, 10)), hi, k)
    else:
        a = math.sqrt(n)
        dims = (max(16, round(a * r)), max(16, round(a / r)))
    if lattice == "honeycomb":
        dims = (dims[0] // 2 * 2, dims[1] // 2 * 2)
    return _case("", op, lattice, dims, B=B, M=M, W=round(rng.uniform(0.5, 8.0), 3), hop=hop, n_t=n_t, dt=dt,
                 nE=rng.randint(101, 1201) if op in ("dos", "train") else 0, tune=rng.random() < 0.75, open_x=open_x,
                 commutator=op == "evolve" and rng.random() < 0.5)


# --------------------------------------------------------------------------- lattices

def _stack(cols):
    return np.ascontiguousarray(np.stack([c.reshape(-1) for c in cols], axis=1).astype(np.int32))


@functools.lru_cache(maxsize=4)
def _neighbours(lattice, Lx, Ly, Lz, open_x):
    """Neighbour list [n, k] (-1: none), counts and x of one lattice, index x + Lx (y + Ly z)."""
    n = Lx * Ly * Lz
    i = np.arange(n, dtype=np.int32).reshape(Lz, Ly, Lx)
    x = np.tile(np.arange(Lx, dtype=np.float64), Ly * Lz)

    def at(dx, dy=0, dz=0):
        return np.roll(i, (-dz, -dy, -dx), (0, 1, 2))

    nn = None
    if lattice == "chain":
        nbr = _stack([at(1), at(-1)])
    elif lattice == "cubic":
        nbr = _stack([at(1), at(-1), at(0, 1), at(0, -1), at(0, 0, 1), at(0, 0, -1)])
    elif lattice == "nnn":
        nbr = _stack([at(1), at(-1), at(0, 1), at(0, -1), at(1, 1), at(-1, 1), at(1, -1), at(-1, -1)])
    elif lattice == "honeycomb":
        up = ((np.arange(Lx)[None, :] + np.arange(Ly)[:, None]) % 2 == 0)[None]
        nbr = _stack([at(1), at(-1), np.where(up, at(0, 1), at(0, -1))])
        x = x * (math.sqrt(3.0) / 2.0 * 0.142)
    elif open_x:
        left, right = at(-1), at(1)
        first = np.broadcast_to(np.arange(Lx) == 0, i.shape)
        last = np.broadcast_to(np.arange(Lx) == Lx - 1, i.shape)
        nbr = _stack([at(0, 1), at(0, -1), np.where(last, left, right), np.where(first | last, -1, left)])
        nn = (4 - (first | last).reshape(-1).astype(np.int32)).astype(np.int32)
    else:
        nbr = _stack([at(1), at(-1), at(0, 1), at(0, -1)])
    if nn is None:
        nn = np.full(n, nbr.shape[1], dtype=np.int32)
    return nbr, nn, x


def _sides(c):
    """Sides of the segments of a `squares` lattice, spaced geometrically."""
    lo, hi, k = c["Lx"], c["Ly"], c["Lz"]
    return [int(round(lo * (hi / lo) ** (r / (k - 1)))) for r in range(k)]


def _hoppings(c, nbr, rng):
    """Hopping of every entry, or None (the default -1)."""
    Lx, Ly = c["Lx"], c["Ly"]
    n, k = nbr.shape
    if c["lattice"] == "nnn":
        h = np.full((n, k), -1.0)
        h[:, 4:] = -0.1
        return h
    t = -2.7 if c["lattice"] == "honeycomb" else -1.0
    if c["hop"] == "entries":
        # one complex number per bond: the +x bond of each row and its +y (or slot 2) bond
        b = [t * (1 + 0.2 * rng.uniform(-1, 1, n)) * np.exp(1j * rng.uniform(-0.3, 0.3, n)) for _ in range(2)]
        h = np.empty((n, k), dtype=np.complex128)
        h[:, 0], h[:, 1] = b[0], np.conj(b[0][nbr[:, 1]])
        if c["lattice"] == "honeycomb":
            up = ((np.arange(Lx)[None, :] + np.arange(Ly)[:, None]) % 2 == 0).reshape(-1)
            h[:, 2] = np.where(up, b[1], np.conj(b[1][nbr[:, 2]]))
        else:
            h[:, 2], h[:, 3] = b[1], np.conj(b[1][nbr[:, 3]])
        return h
    if c["lattice"] != "honeycomb":
        return None
    if c["hop"] != "flux":
        return np.full((n, k), t)
    # Peierls phases of `q` flux quanta through the sample
    q = max(1, Lx * Ly // 4000)
    flux = 2.0 * q / (Lx * Ly)
    i, j = np.arange(n) % Lx, np.arange(n) // Lx
    th = -math.pi * flux * j
    up = (i + j) % 2 == 0
    h = np.empty((n, k), dtype=np.complex128)
    h[:, 0], h[:, 1], h[:, 2] = t * np.exp(-1j * th), t * np.exp(1j * th), t
    w = math.pi * flux * Ly * i
    h[:, 2] = np.where(up & (j == Ly - 1), t * np.exp(-1j * w), h[:, 2])
    h[:, 2] = np.where(~up & (j == 0), t * np.exp(1j * w), h[:, 2])
    return h


def _band(c):
    """Half width of the spectrum without disorder, and of the disorder."""
    per = {"chain": 2.0, "cubic": 6.0, "honeycomb": 8.1, "nnn": 4.4}.get(c["lattice"], 4.0)
    return per * (1.2 if c["hop"] == "entries" else 1.0), 0.5 * c["W"]


def _model(c, seed):
    """The descriptor arrays of a case, on the host."""
    rng = np.random.default_rng(seed)
    m = dict(energy_max=1.01 * sum(_band(c)), volume=1.0)
    if c["lattice"] == "squares":
        parts = [_neighbours("square", s, s, 1, False) for s in _sides(c)]
        off = np.cumsum([0] + [p[0].shape[0] for p in parts])
        m.update(nbr=np.concatenate([p[0] + o for p, o in zip(parts, off.astype(np.int32))]),
                 nn=np.concatenate([p[1] for p in parts]), x=np.concatenate([p[2] for p in parts]), length_x=0.0,
                 seg_offsets=off, seg_length_x=[float(s) for s in _sides(c)],
                 seg_energy_max=[m["energy_max"]] * len(parts))
    else:
        nbr, nn, x = _neighbours(c["lattice"], c["Lx"], c["Ly"], c["Lz"], c["open_x"])
        length = 0.0 if c["open_x"] else c["Lx"] * (math.sqrt(3.0) / 2.0 * 0.142 if c["lattice"] == "honeycomb" else 1.0)
        m.update(nbr=nbr, nn=nn, x=x, length_x=length)
        m["hop"] = _hoppings(c, nbr, rng)
        if c["lattice"] == "nnn":
            cls = np.zeros(nbr.shape, dtype=np.int32)
            cls[:, 4:] = 1
            m.update(hop_class=cls, n_class=2)
    n = m["nn"].shape[0]
    m["onsite"] = rng.random(n) * c["W"] - 0.5 * c["W"]
    m["volume"] = float(n)
    return m


def _phases(n, B, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    th = torch.rand((n, B), generator=g, device="cuda", dtype=torch.float64) * (2.0 * math.pi)
    return torch.polar(torch.ones_like(th), th)


def _inputs(c, n, seed):
    """Vectors and loss weights of a case, on the GPU."""
    s = dict(phi=_phases(n, c["B"], 7919 * seed + 1))
    if c["commutator"]:
        s["chi"] = _phases(n, c["B"], 7919 * seed + 2)
    e = _band(c)[0] * 0.95
    s["E"] = np.linspace(-e, e, c["nE"])
    s["dt"] = [c["dt"] * (1 + 0.25 * k) for k in range(c["n_t"])]
    g = torch.Generator(device="cuda").manual_seed(7919 * seed + 3)
    if c["op"] == "train":
        s["target"] = torch.rand((1, c["nE"]), generator=g, device="cuda", dtype=torch.float64) * 0.2
        s["w"] = torch.randn((c["n_t"], 1, 1, c["M"]), generator=g, device="cuda", dtype=torch.float64) / c["M"]
    if c["op"] == "bonds":
        s["w"] = torch.randn((1, c["B"], c["M"]), generator=g, device="cuda", dtype=torch.float64)
    return s


# --------------------------------------------------------------------------- a user's program

def prepare(case, seed):
    c = case
    m = _model(c, seed)
    s = _inputs(c, m["nn"].shape[0], seed)
    h = P.gpuqt_build_h(**m, no_dictionary=c["lattice"] == "honeycomb" and c["hop"] == "entries")
    if c["tune"]:
        P.gpuqt_autotune_cached(h, c["B"])
    if c["op"] == "train":
        s["onsite"] = torch.from_numpy(m["onsite"]).cuda().requires_grad_(True)
        s["scales"] = torch.ones(2, dtype=torch.float64, device="cuda").requires_grad_(True)
    s.update(c=c, H=h, energy_max=m["energy_max"], volume=m["volume"], k=m["nbr"].shape[1])
    return s


def run(state):
    s, c, h = state, state["c"], state["H"]
    if c["op"] == "dos":
        mu = P.gpuqt_moments(h, s["phi"], s["phi"], c["M"])
        rows = mu.real.reshape(-1, c["M"]).contiguous()
        return {"mu": mu, "rho": P.gpuqt_kpm_reconstruct(rows, s["E"], s["energy_max"], s["volume"])}
    if c["op"] == "vac":
        return P.gpuqt_vac(h, s["phi"], s["dt"], c["M"], c["Np"])
    if c["op"] == "msd":
        return P.gpuqt_msd(h, s["phi"], s["dt"], c["M"], c["Np"])
    if c["op"] == "evolve":
        return P.gpuqt_evolve(h, s["phi"], c["dt"], c["Np"], chi=s.get("chi"), with_commutator=c["commutator"])
    if c["op"] == "train":
        s["onsite"].grad = s["scales"].grad = None
        mu = A.Moments.apply(s["onsite"], s["scales"], h, s["phi"], c["M"])
        rho = A.KPM.apply(mu.reshape(1, c["M"]), s["E"], s["energy_max"], s["volume"])
        vac = A.VAC.apply(s["onsite"], s["scales"], h, s["phi"], s["dt"], c["M"], c["Np"])
        loss = ((rho - s["target"]) ** 2).sum() + (s["w"] * vac).sum()
        loss.backward()
        return {"loss": loss.detach(), "rho": rho.detach(), "vac": vac.detach(), "d_onsite": s["onsite"].grad,
                "d_scales": s["scales"].grad}
    n = s["phi"].shape[0]
    gu = torch.zeros(n, dtype=torch.float64, device="cuda")
    gh = torch.zeros((n, s["k"], 2), dtype=torch.float64, device="cuda")
    P.gpuqt_moments_backward(h, s["phi"], s["phi"], s["w"], grad_onsite=gu, grad_hop=gh)
    return {"d_onsite": gu, "d_hop": gh}


# --------------------------------------------------------------------------- size of the work

def _rows(c):
    return sum(v * v for v in _sides(c)) if c["lattice"] == "squares" else c["Lx"] * c["Ly"] * c["Lz"]


def _terms(c, dt):
    return c["Np"] or int(1.01 * sum(_band(c)) * dt) + 20


def work(case):
    c = case
    n, B, M = _rows(c), c["B"], c["M"]
    k = {"chain": 2, "honeycomb": 3, "cubic": 6, "nnn": 8}.get(c["lattice"], 4)
    cplx = c["hop"] in ("flux", "entries")
    step = n * B * ((8 if cplx else 4) * k + 12)     # one sparse product with its combine, in flops
    dots = 8 * n * B
    dts = [c["dt"] * (1 + 0.25 * j) for j in range(c["n_t"])]
    vec, vin, out = 16 * n * B, 1, 0
    if c["op"] == "dos":
        flops = M // 2 * (step + 2 * dots)
        out = 16 * B * M * (c["Lz"] if c["lattice"] == "squares" else 1) + 8 * B * c["nE"]
    elif c["op"] == "vac":
        flops = c["n_t"] * M // 2 * (2 * step + 2 * dots) + sum(2 * _terms(c, t) * (step + 4 * n * B) for t in dts[:-1])
        out = 8 * c["n_t"] * B * M
    elif c["op"] == "msd":
        flops = c["n_t"] * M // 2 * (step + 2 * dots) + sum(_terms(c, t) * 2 * (1.3 * step + 4 * n * B) for t in dts)
        out = 8 * c["n_t"] * B * M
    elif c["op"] == "evolve":
        q = 2 if c["commutator"] else 1
        flops, vin, out = _terms(c, c["dt"]) * q * (step + 4 * n * B), q, q * vec
    elif c["op"] == "train":
        rows = M // 2 * (1 + 2 * c["n_t"]) + 2 * sum(_terms(c, t) for t in dts[:-1])
        flops, out = 3 * rows * (step + 2 * dots), 8 * n + 8 * c["n_t"] * M + 8 * c["nE"]
    else:
        flops, out = 2 * M * step + M * 8 * n * B * k, 8 * n + 16 * n * k
    matrix = n * (8 + (20 if c["hop"] == "entries" else 4) * k)
    return {"bytes": matrix + vin * vec + out, "flops": flops}


# --------------------------------------------------------------------------- the same in plain torch

class _Plain:
    """H / energy_max, the commutator and the velocity of a case's model on [n, B] tensors."""

    def __init__(self, m):
        self.dE = m["energy_max"]
        nbr = torch.from_numpy(m["nbr"]).cuda().long()
        self.pad = None if int(m["nn"].min()) == nbr.shape[1] else nbr < 0
        self.nbr = [q.contiguous() for q in nbr.clamp(min=0).unbind(1)]
        hop = m.get("hop")
        self.hop = None if hop is None else torch.from_numpy(hop).cuda() / self.dE
        self.diag = torch.from_numpy(m["onsite"]).cuda()[:, None] / self.dE
        self.x, self.length, self.m = torch.from_numpy(m["x"]).cuda(), m["length_x"], m
        self.dx = None
        self.scales = None

    def weight(self, s):
        if self.hop is not None:
            w = self.hop[:, s, None]
        elif self.pad is not None:
            w = (~self.pad[:, s, None]).double() * (-1.0 / self.dE)
        else:
            w = -1.0 / self.dE
        return w if self.scales is None else w * self.scales[0 if s < 4 else 1]

    def H(self, v):
        out = self.diag * v
        if self.hop is None and self.pad is None:
            t = v.index_select(0, self.nbr[0])
            for q in self.nbr[1:]:
                t += v.index_select(0, q)
            return out.add_(t, alpha=-1.0 / self.dE)
        for s, q in enumerate(self.nbr):
            out = out + self.weight(s) * v.index_select(0, q)
        return out

    def dH(self, v):
        """sum_j (x_j - x_i) (H / energy_max)_ij v_j."""
        out = torch.zeros_like(v)
        for s, q in enumerate(self.nbr):
            d = self.x[q] - self.x
            if "seg_length_x" in self.m:
                off = self.m["seg_offsets"]
                L = torch.repeat_interleave(torch.tensor(self.m["seg_length_x"], device="cuda", dtype=torch.float64),
                                            torch.from_numpy(np.diff(off)).cuda())
                d = d - L * torch.round(d / L)
            elif self.length > 0:
                d = d - self.length * torch.round(d / self.length)
            out = out + (d[:, None] * self.weight(s)) * v.index_select(0, q)
        return out

    def V(self, v):
        return 1j * self.dE * self.dH(v)

    def XH(self, v):
        return -self.dH(v)


def _dot(a, b, off):
    """<a|b> per segment and column."""
    if off is None:
        return (a.conj() * b).sum(0)[None]
    p = a.conj() * b
    return torch.stack([p[lo:hi].sum(0) for lo, hi in zip(off[:-1], off[1:])])


def _moments(H, a, b, M, off=None):
    """<a|T_n|b>, [segments, B, M], through T_2k = 2 T_k T_k - 1 and T_2k+1 = 2 T_k+1 T_k - T_1."""
    mu = [_dot(a, b, off), _dot(a, H(b), off)]
    same = a is b
    a0, a1 = a, H(a)
    b0, b1 = (a0, a1) if same else (b, H(b))
    while len(mu) < M:
        mu.append(2 * _dot(a1, b1, off) - mu[0])
        a0, a1 = a1, 2 * H(a1) - a0
        b0, b1 = (a0, a1) if same else (b1, 2 * H(b1) - b0)
        mu.append(2 * _dot(a1, b0, off) - mu[1])
    return torch.stack(mu[:M], dim=-1)


def _bessel(tau, n):
    """J_0 .. J_{n-1} of tau by the trapezoid rule on their integral, exact to rounding here."""
    q = 4 * (n + int(abs(tau)) + 64)
    th = torch.arange(q, device="cuda", dtype=torch.float64) * (2 * math.pi / q)
    m = torch.arange(n, device="cuda", dtype=torch.float64)[:, None]
    return torch.cos(m * th - tau * torch.sin(th)).mean(1).tolist()


def _series(p, psi, dt, Np, chi=None, with_chi=False):
    """U(dt) psi and, with_chi, [X, U(dt)] psi + U(dt) chi."""
    tau = p.dE * abs(dt)
    J = _bessel(tau, (Np or int(tau) + 60 + int(12 * (tau + 1) ** (1 / 3))))
    ph = -1j if dt >= 0 else 1j
    a0, a1 = psi, p.H(psi)
    out = J[0] * a0 + 2 * ph * J[1] * a1
    if with_chi:
        b0 = torch.zeros_like(psi) if chi is None else chi
        b1 = p.XH(a0) + p.H(b0)
        oc = J[0] * b0 + 2 * ph * J[1] * b1
    for m in range(2, len(J)):
        if with_chi:
            b0, b1 = b1, 2 * p.XH(a1) + 2 * p.H(b1) - b0
        a0, a1 = a1, 2 * p.H(a1) - a0
        f = 2 * ph ** m * J[m]
        out = out + f * a1
        if with_chi:
            oc = oc + f * b1
    return (out, oc) if with_chi else out


def _kpm(mu, E, dE, volume):
    """Jackson-damped KPM sums of rows [R, M] on the energies E."""
    M = mu.shape[-1]
    n = torch.arange(M, device="cuda", dtype=torch.float64)
    a = 1.0 / (M + 1)
    g = (1 - n * a) * torch.cos(math.pi * n * a) + a * torch.sin(math.pi * n * a) / math.tan(math.pi * a)
    x = torch.from_numpy(E).cuda() / dE
    t = torch.cos(n[:, None] * torch.acos(x)) * (g * torch.where(n == 0, 1.0, 2.0))[:, None]
    return mu @ t * (2.0 / (math.pi * volume * dE)) / torch.sqrt(1 - x * x)


def exact(case, seed):
    c = case
    m = _model(c, seed)
    s = _inputs(c, m["nn"].shape[0], seed)
    p = _Plain(m)
    phi, M, dts = s["phi"], c["M"], s["dt"]
    off = None if "seg_offsets" not in m else [int(v) for v in m["seg_offsets"]]
    if c["op"] == "dos":
        mu = _moments(p.H, phi, phi, M, off)
        return {"mu": mu, "rho": _kpm(mu.real.reshape(-1, M), s["E"], p.dE, m["volume"])}
    if c["op"] == "evolve":
        return _series(p, phi, c["dt"], c["Np"], s.get("chi"), c["commutator"])
    if c["op"] == "vac":
        left, right, rows = phi, p.V(phi), []
        for k in range(c["n_t"]):
            rows.append(_moments(p.H, p.V(left), right, M, off).real)
            if k + 1 < c["n_t"]:
                left, right = _series(p, left, -dts[k], c["Np"]), _series(p, right, -dts[k], c["Np"])
        return torch.stack(rows)
    if c["op"] == "msd":
        psi, chi, rows = phi, None, []
        for k in range(c["n_t"]):
            psi, chi = _series(p, psi, dts[k], c["Np"], chi, True)
            rows.append(_moments(p.H, chi, chi, M, off).real)
        return torch.stack(rows)
    if c["op"] == "train":
        return _exact_train(c, m, s, p)
    # bonds: the reverse of the plain recurrence, every forward vector kept
    w = s["w"][0]
    v = [phi, p.H(phi)]
    while len(v) < M:
        v.append(2 * p.H(v[-1]) - v[-2])
    gu = torch.zeros(phi.shape[0], dtype=torch.float64, device="cuda")
    gh = torch.zeros((phi.shape[0], len(p.nbr)), dtype=C128, device="cuda")
    l1 = l2 = torch.zeros_like(phi)
    for n in range(M - 1, 0, -1):
        lam = w[:, n] * phi + 2 * p.H(l1) - l2
        f = (1.0 if n == 1 else 2.0) / p.dE
        gu += f * (lam.conj() * v[n - 1]).real.sum(1)
        for q, nb in enumerate(p.nbr):
            gh[:, q] += f * (lam.conj() * v[n - 1][nb]).sum(1)
        l1, l2 = lam, l1
    return {"d_onsite": gu, "d_hop": torch.view_as_real(gh.conj().resolve_conj())}


def _exact_train(c, m, s, p):
    from torch.utils.checkpoint import checkpoint

    onsite = torch.from_numpy(m["onsite"]).cuda().requires_grad_(True)
    scales = torch.ones(2, dtype=torch.float64, device="cuda").requires_grad_(True)
    Lx, Ly, M = c["Lx"], c["Ly"], c["M"]
    shifts = [(1, 0), (-1, 0), (0, 1), (0, -1), (1, 1), (-1, 1), (1, -1), (-1, -1)]
    t = [-1.0 / p.dE, -0.1 / p.dE]

    def H(v):
        g = v.view(Ly, Lx, -1)
        r = [sum(torch.roll(g, (-dy, -dx), (0, 1)) for dx, dy in q) for q in (shifts[:4], shifts[4:])]
        return (onsite / p.dE)[:, None] * v + (scales[0] * t[0] * r[0] + scales[1] * t[1] * r[1]).view_as(v)

    def V(v):
        g = v.view(Ly, Lx, -1)
        r = [sum(dx * torch.roll(g, (-dy, -dx), (0, 1)) for dx, dy in q if dx) for q in (shifts[:4], shifts[4:])]
        return 1j * p.dE * (scales[0] * t[0] * r[0] + scales[1] * t[1] * r[1]).view_as(v)

    class Q:
        dE = p.dE

    Q.H = staticmethod(H)
    phi = s["phi"]
    mu = checkpoint(lambda: _moments(H, phi, phi, M).real, use_reentrant=False)
    rho = _kpm(mu.reshape(1, M), s["E"], p.dE, m["volume"])
    left, right, rows = phi, V(phi), []
    for k in range(c["n_t"]):
        rows.append(checkpoint(lambda a, b: _moments(H, V(a), b, M).real, left, right, use_reentrant=False))
        if k + 1 < c["n_t"]:
            step = functools.partial(_series, Q, dt=-s["dt"][k], Np=c["Np"])
            left = checkpoint(step, left, use_reentrant=False)
            right = checkpoint(step, right, use_reentrant=False)
    vac = torch.stack(rows)
    loss = ((rho - s["target"]) ** 2).sum() + (s["w"] * vac).sum()
    loss.backward()
    return {"loss": loss.detach(), "rho": rho.detach(), "vac": vac.detach(), "d_onsite": onsite.grad,
            "d_scales": scales.grad}
