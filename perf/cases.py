"""Performance cases of the library: what a user runs, over the sizes they run it at.

Three kinds of cell, built here from a seed (bond springs of a central pair
potential, masses and springs drawn a few percent around the usual values):
the two-atom diamond cell, the five-atom cubic ABX3 cell (both on Gamma-centred
meshes) and displaced-diamond glasses at the Gamma point.  A case is one
pass of a workflow over them:

  run     phonons, linewidths of every mode, RTA conductivity (the whole call)
  modes   linewidths of every mode from phonons in hand, optionally with
          isotope scattering added, and the conductivity
  wedge   linewidths of the irreducible wedge, mapped to the full mesh
  glass   linewidths of a Gamma-point solid, optionally its QHGK conductivity
  bte     scattering matrix and its direct inversion
  sweep   temperature cache and linewidths at 16 temperatures
"""
from __future__ import annotations

import itertools
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_2602_23728_amd import kaldo as K
from paper_2602_23728_amd import learned

PREC = {"fp64": K.FP64, "fp32": K.FP32, "bf16x3": K.BF16X3}
SHAPE = {"gauss": K.GAUSS, "lorentz": K.LORENTZ}
NU_MIN, SIGMA, FLOOR = 0.1, 0.1, 0.01  # THz: frequency floor, fixed width, smallest adaptive width
G_SILICON, G_LEAD = 2.007e-4, 4.94e-5  # natural isotope mass variances
SWEEP_T = tuple(float(t) for t in np.linspace(100.0, 850.0, 16))

# CODATA 2018, in eV, Angstrom, amu, ps, K
EV, AMU, HBAR_J, KB_J = 1.602176634e-19, 1.66053906660e-27, 1.054571817e-34, 1.380649e-23
HBAR, KB = HBAR_J / EV * 1e12, KB_J / EV
UNIT = EV / (1e-20 * AMU) * 1e-24
TWO_PI = 2.0 * math.pi
KAPPA_UNIT = KB_J * 1e4 * 1e-12 / 1e-30


def _case(name, kind, cell, n1, n2, n3, precision, *, shape="gauss", adaptive=True, kelvin=300.0,
          extra=False):
    c = dict(kind=kind, cell=cell, n1=n1, n2=n2, n3=n3, precision=precision, shape=shape,
             adaptive=adaptive, kelvin=kelvin, extra=extra)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest whole run: a quick look at a cell, where launches and latency count
        _case("run-diamond-5-fp64", "run", "diamond", 5, 5, 5, "fp64", adaptive=False),
        # the production run: a converged mesh in the precision the method is published in
        _case("run-diamond-24-fp64", "run", "diamond", 24, 24, 24, "fp64"),
        # a convergence study's mesh in FP32, natural silicon's isotopes added (extra)
        _case("modes-diamond-15-fp32", "modes", "diamond", 15, 15, 15, "fp32", extra=True),
        # the converged mesh by symmetry: 413 of its 13,824 q-points
        _case("wedge-diamond-24-fp32", "wedge", "diamond", 24, 24, 24, "fp32"),
        # a larger cell on a converged mesh, FP32 on the matrix cores
        _case("modes-abx3-12-fp32", "modes", "abx3", 12, 12, 12, "fp32"),
        # the same cell in split precision, on an anisotropic mesh of odd extents
        _case("modes-abx3-11x9x7-bf16x3", "modes", "abx3", 11, 9, 7, "bf16x3", kelvin=500.0),
        # the same cell in FP64, Lorentzian of fixed width, a small mesh of unequal extents
        _case("modes-abx3-7x6x5-fp64", "modes", "abx3", 7, 6, 5, "fp64", shape="lorentz",
              adaptive=False),
        # a 512-atom glass in FP32 with the QHGK conductivity it is computed for (extra)
        _case("glass-512-fp32-qhgk", "glass", "glass", 4, 4, 4, "fp32", adaptive=False, extra=True),
        # split precision on a cell of 384 atoms
        _case("glass-384-bf16x3", "glass", "glass", 4, 4, 3, "bf16x3", adaptive=False),
        # FP64 on a cell of 216 atoms
        _case("glass-216-fp64", "glass", "glass", 3, 3, 3, "fp64", adaptive=False),
        # the linearised transport equation beyond the relaxation-time approximation
        _case("bte-diamond-15", "bte", "diamond", 15, 15, 15, "fp64"),
        # conductivity against temperature: the factors once, then 16 temperatures
        _case("sweep-diamond-20-fp64", "sweep", "diamond", 20, 20, 20, "fp64"),
    ]


def _mesh_draw(rng, lo, hi):
    """Extents of a mesh of lo^3 to hi^3 points, spread over the logarithm, a little unequal."""
    n = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    dims = [max(lo - 1, min(hi, round(n * rng.uniform(0.85, 1.15)))) for _ in range(3)]
    return dims


def draw(rng):
    kind = rng.choice(["run", "modes", "modes", "wedge", "glass", "glass", "bte", "sweep"])
    kelvin = float(rng.randint(10, 90) * 10)
    if kind == "run":
        return _case(None, kind, "diamond", *_mesh_draw(rng, 5, 23), "fp64",
                     adaptive=rng.random() < 0.7, kelvin=kelvin)
    if kind == "modes":
        adaptive = rng.random() < 0.7
        shape = rng.choice(["gauss", "gauss", "lorentz"])
        if rng.random() < 0.4:
            return _case(None, kind, "diamond", *_mesh_draw(rng, 5, 16), rng.choice(["fp64", "fp32"]),
                         shape=shape, adaptive=adaptive, kelvin=kelvin, extra=rng.random() < 0.5)
        precision = rng.choice(["fp64", "fp32", "bf16x3"])
        return _case(None, kind, "abx3", *_mesh_draw(rng, 4, 7 if precision == "fp64" else 11),
                     precision, shape=shape, adaptive=adaptive, kelvin=kelvin,
                     extra=rng.random() < 0.3)
    if kind == "wedge":
        n = rng.randint(6, 23)
        return _case(None, kind, "diamond", n, n, n, rng.choice(["fp64", "fp32"]), kelvin=kelvin)
    if kind == "glass":
        precision = rng.choice(["fp64", "fp32", "bf16x3"])
        top = 3 if precision == "fp64" else 4
        dims = [rng.randint(2, top) for _ in range(3)]
        return _case(None, kind, "glass", *dims, precision, shape=rng.choice(["gauss", "lorentz"]),
                     adaptive=False, kelvin=kelvin, extra=rng.random() < 0.4)
    if kind == "bte":
        return _case(None, kind, "diamond", *_mesh_draw(rng, 4, 14), "fp64", kelvin=kelvin)
    return _case(None, kind, "diamond", *_mesh_draw(rng, 6, 19), rng.choice(["fp64", "fp32"]),
                 kelvin=kelvin)


# ------------------------------------------------------------------ cells

def _pair_blocks(n, r0, k2, k3):
    """Second and third derivatives of k2/2 (r-r0)^2 + k3/6 (r-r0)^3 at r0, n the unit vector."""
    eye = np.eye(3)
    t3 = (k3 - 3.0 * k2 / r0) * np.einsum("a,b,c->abc", n, n, n)
    t3 += (k2 / r0) * (np.einsum("ab,c->abc", eye, n) + np.einsum("ac,b->abc", eye, n)
                       + np.einsum("bc,a->abc", eye, n))
    return k2 * np.outer(n, n), t3


def _cell(lattice, frac, mass, rep, bonds):
    """FC2 and COO FC3 from bonds (i, replica, j, vector, k2, k3) with i in the home cell."""
    nb, nr = len(mass), len(rep)
    fc2 = np.zeros((3 * nb, nr, 3 * nb))
    third = {}
    for i, l, j, d, k2, k3 in bonds:
        r0 = float(np.linalg.norm(d))
        t2, t3 = _pair_blocks(d / r0, r0, k2, k3)
        fc2[3 * i:3 * i + 3, l, 3 * j:3 * j + 3] -= t2
        fc2[3 * i:3 * i + 3, 0, 3 * i:3 * i + 3] += t2
        a, b = i, l * nb + j
        for s2, s3 in itertools.product((a, b), (a, b)):
            sign = -1.0 if (s2 == a) == (s3 == a) else 1.0
            third[i, s2, s3] = third.get((i, s2, s3), 0.0) + sign * t3
    keys = np.array(sorted(third))
    blocks = np.stack([third[tuple(k)] for k in keys])
    axis = np.indices((3, 3, 3)).reshape(3, -1)
    ijk = [(3 * keys[:, c, None] + axis[c][None, :]).reshape(-1).astype(np.int32) for c in range(3)]
    return SimpleNamespace(lattice=lattice, frac=frac, mass=mass, rep=rep, fc2=fc2, n_basis=nb,
                           fc3_i=ijk[0], fc3_j=ijk[1], fc3_k=ijk[2], fc3_val=blocks.reshape(-1),
                           volume=float(abs(np.linalg.det(lattice))))


def _replicas():
    r = [c for c in itertools.product((-1, 0, 1), repeat=3) if c != (0, 0, 0)]
    return np.array([(0, 0, 0)] + r, np.int32)


def _near(lattice, frac, rep, cutoff):
    cart = frac @ lattice
    for i in range(len(frac)):
        for l, r in enumerate(rep):
            for j in range(len(frac)):
                d = r @ lattice + cart[j] - cart[i]
                if (l or j != i) and np.linalg.norm(d) < cutoff:
                    yield i, l, j, d


def _build(case, seed):
    rng = np.random.default_rng(seed)
    around = lambda x, rel=0.05: float(x * rng.uniform(1.0 - rel, 1.0 + rel))  # noqa: E731
    if case["cell"] == "diamond":
        a, m, k2, k3 = 5.43, around(28.085), around(10.0), around(-60.0)
        lat = 0.5 * a * np.array([[0, 1, 1], [1, 0, 1], [1, 1, 0]], float)
        frac = np.array([[0, 0, 0], [0.25, 0.25, 0.25]])
        rep = _replicas()
        return _cell(lat, frac, np.array([m, m]), rep,
                     [(*b, k2, k3) for b in _near(lat, frac, rep, 3.0)])
    if case["cell"] == "abx3":
        lat = 6.3 * np.eye(3)
        frac = np.array([[0, 0, 0], [0.5, 0.5, 0.5], [0.5, 0.5, 0], [0.5, 0, 0.5], [0, 0.5, 0.5]])
        species = "ABXXX"
        mass = np.array([around(133.0), around(207.0)] + [around(127.0)] * 3)
        spring = {t: (around(k2), around(k3)) for t, k2, k3 in
                  (("AX", 5.8, -39.5), ("BX", 3.6, -15.6), ("XX", 2.2, -12.6))}
        rep = _replicas()
        bonds = []
        for b in _near(lat, frac, rep, 4.5):
            t = "".join(sorted(species[b[0]] + species[b[2]]))
            if t in spring:
                bonds.append((*b, *spring[t]))
        return _cell(lat, frac, mass, rep, bonds)
    basis = np.array([[0, 0, 0], [0, 2, 2], [2, 0, 2], [2, 2, 0],
                      [1, 1, 1], [1, 3, 3], [3, 1, 3], [3, 3, 1]]) / 4.0
    n = np.array([case["n1"], case["n2"], case["n3"]])
    box = 5.43 * n
    cells = np.array(list(itertools.product(*(range(x) for x in n))), float)
    pos = 5.43 * (cells[:, None, :] + basis[None]).reshape(-1, 3)
    pos = pos + rng.normal(0.0, 0.08, pos.shape)
    d = pos[None] - pos[:, None]
    d -= box * np.round(d / box)
    near = np.argwhere((np.einsum("ijk,ijk->ij", d, d) < 2.8 ** 2) & ~np.eye(len(pos), dtype=bool))
    # a bond seen from both ends: FC3's first index runs over every atom of the one cell
    k2, k3, m = around(10.0), around(-60.0), around(28.085)
    return _cell(np.diag(box), pos / box, np.full(len(pos), m), np.zeros((1, 3), np.int32),
                 [(i, 0, j, d[i, j], k2, k3) for i, j in near])


# ------------------------------------------------------------------ phonons in hand

def _mesh(case):
    return (case["n1"], case["n2"], case["n3"]) if case["cell"] != "glass" else (1, 1, 1)


def _points(mesh):
    return np.stack(np.meshgrid(*(np.arange(n) for n in mesh), indexing="ij"), -1).reshape(-1, 3)


def _phonons(m, mesh):
    """omega [nq, n], eta [nq, n, n] (component, mode), v [nq, n, 3] in 64 bits on the host."""
    phase = np.exp(-1j * TWO_PI * ((_points(mesh) / np.array(mesh)) @ m.rep.T))
    dof = np.repeat(m.mass, 3)
    inv = 1.0 / np.sqrt(np.outer(dof, dof))
    n = len(dof)
    fc = m.fc2.transpose(1, 0, 2).reshape(len(m.rep), -1)
    D = (phase @ fc).reshape(-1, n, n) * inv
    lam, eta = np.linalg.eigh(0.5 * (D + D.conj().transpose(0, 2, 1)))
    omega = np.sign(lam) * np.sqrt(np.abs(lam) * UNIT)
    vel = np.zeros((*omega.shape, 3))
    ok = omega >= TWO_PI * 1e-3
    R = m.rep @ m.lattice
    for c in range(3):
        dD = ((phase * (-1j * R[:, c])) @ fc).reshape(-1, n, n) * inv
        g = np.real(np.sum(eta.conj() * (dD @ eta), axis=1))
        vel[..., c][ok] = g[ok] * UNIT / (2.0 * omega[ok])
    return omega, eta, vel


def _glass_modes(m):
    dof = np.repeat(m.mass, 3)
    D = torch.from_numpy(m.fc2[:, 0, :] / np.sqrt(np.outer(dof, dof)))
    lam, E = torch.linalg.eigh(0.5 * (D + D.T))
    return (lam.sign() * (lam.abs() * UNIT).sqrt()).numpy(), E.numpy()


def _cuda(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _broadening(case):
    return SimpleNamespace(shape=SHAPE[case["shape"]], adaptive=case["adaptive"], sigma_thz=SIGMA,
                           sigma_floor_thz=FLOOR, nu_min_thz=NU_MIN)


def _g_factor(case):
    return [G_SILICON] * 2 if case["cell"] == "diamond" else [0.0, G_LEAD, 0.0, 0.0, 0.0]


def prepare(case, seed):
    """The crystal handle, phonons where the workflow has them in hand, and the workspaces a
    program keeps between calls."""
    m = _build(case, seed)
    mesh, prec = _mesh(case), PREC[case["precision"]]
    s = SimpleNamespace(case=case, mesh=mesh, prec=prec, b=_broadening(case), frac=m.frac,
                        c=K.Crystal.from_model(m), T=case["kelvin"], g=_g_factor(case))
    buf = lambda n: torch.empty(max(int(n), 1), dtype=torch.uint8, device="cuda")  # noqa: E731
    kind = case["kind"]
    if kind == "glass":
        s.omega, s.evec = (_cuda(x) for x in _glass_modes(m))
        s.ws = buf(K.lib().kaldo_linewidths_gamma_workspace(s.c.handle, prec))
        return s
    if kind == "bte":
        s.omega, s.evec, s.vel = K.phonons(s.c, mesh)
        s.ws = buf(K.bte_workspace(s.c, mesh))
        n = s.omega.numel()
        s.matrix = (torch.empty(n, n, dtype=torch.float64, device="cuda"),
                    torch.empty(n, dtype=torch.float64, device="cuda"))
        return s
    if kind != "run":
        s.omega, s.evec, s.vel = (_cuda(x) for x in _phonons(m, mesh))
    if kind == "sweep":
        s.ws = buf(K.tcache_workspace(s.c, mesh, prec))
        return s
    if kind == "wedge":
        s.wedge = learned.Wedge(m.lattice, m.frac, m.mass, mesh)
    s.ws = buf(K.linewidths_workspace(s.c, mesh, prec))
    return s


def run(s):
    kind = s.case["kind"]
    if kind == "glass":
        gamma = K.linewidths_gamma(s.c, s.omega, s.evec, s.T, s.b, s.prec, workspace=s.ws)
        if not s.case["extra"]:
            return {"gamma": gamma}
        kappa, diff = K.qhgk_gamma(s.c, s.frac, s.omega, s.evec, gamma, s.T, NU_MIN)
        return {"gamma": gamma, "kappa": kappa, "diffusivity": diff}
    if kind == "bte":
        matrix, gamma0 = K.scattering_matrix(s.c, s.mesh, s.omega, s.evec, s.vel, s.T, s.b,
                                             workspace=s.ws, out=s.matrix)
        lam, kappa = K.bte_solve(s.c, s.mesh, s.omega, s.vel, gamma0, s.T, NU_MIN, matrix,
                                 workspace=s.ws)
        return {"gamma0": gamma0, "lambda": lam, "kappa": kappa}
    if kind == "sweep":
        cache = K.tcache_build(s.c, s.mesh, s.omega, s.evec, s.vel, s.b, s.prec, workspace=s.ws)
        return {"gamma": K.tcache_gamma(s.c, cache, s.omega, NU_MIN, SWEEP_T)}
    if kind == "wedge":
        return {"gamma": learned.plain_ibz_linewidths(s.c, s.wedge, s.omega, s.evec, s.vel, s.T,
                                                      s.b, s.prec)}
    if kind == "run":
        omega, evec, vel = K.phonons(s.c, s.mesh)
        gamma = K.linewidths(s.c, s.mesh, omega, evec, vel, s.T, s.b, s.prec, workspace=s.ws)
        kappa = K.kappa_rta(s.c, s.mesh, omega, vel, gamma, s.T, NU_MIN)
        return {"omega": omega, "evec": evec, "vel": vel, "gamma": gamma, "kappa": kappa}
    gamma = K.linewidths(s.c, s.mesh, s.omega, s.evec, s.vel, s.T, s.b, s.prec, workspace=s.ws)
    if s.case["extra"]:
        K.isotope_linewidths(s.c, s.mesh, s.omega, s.evec, s.vel, s.g, s.b, out=gamma,
                             accumulate=True)
    kappa = K.kappa_rta(s.c, s.mesh, s.omega, s.vel, gamma, s.T, NU_MIN)
    return {"gamma": gamma, "kappa": kappa}


# ------------------------------------------------------------------ work

# Shares of the (mode, partner pair) candidates inside the energy cut, rounded from counts on
# the cells above (diamond 15^3 to 24^3, abx3 12^3), and the distinct FC3 patterns of each cell.
PASS = {"diamond": 0.006, "abx3": 0.01, "glass": 0.05}
PATTERNS = {"diamond": 216, "abx3": 1665}


def work(case):
    """Inputs read once, outputs written once; one energy test per unordered partner pair and the
    projection of the pairs inside the cut.  The inversion counts its LU of two thirds of the
    modes, a glass its sparse product and the live share of its dense one."""
    if case["kind"] == "glass":
        n = 24.0 * case["n1"] * case["n2"] * case["n3"]
        flops = n * (2.0 * 45 * n * n + 2.0 * 0.1 * n ** 3) + (3.0 * n ** 3 if case["extra"] else 0.0)
        return {"bytes": 8.0 * (n * n + 3 * n), "flops": flops}
    nb3 = {"diamond": 6, "abx3": 15}[case["cell"]]
    nq = float(case["n1"] * case["n2"] * case["n3"])
    modes = nq * nb3
    pairs = modes * modes * nb3 / 2
    if case["kind"] == "wedge":
        pairs *= 1.0 / 40 + 2.0 / nq
    flops = 8.0 * pairs + PASS[case["cell"]] * pairs * 8.0 * PATTERNS[case["cell"]]
    size = 8.0 * modes * (1 + 2 * nb3 + 3 + 1)
    if case["kind"] == "bte":
        flops += 2.0 / 3.0 * (2.0 * modes / 3.0) ** 3
        size += 16.0 * modes * modes
    if case["kind"] == "sweep":
        size += 8.0 * modes * len(SWEEP_T)
    return {"bytes": size, "flops": flops}


# ------------------------------------------------------------------ the same in 64 bits

def _bose(w, T):
    return 1.0 / torch.expm1(HBAR * w / (KB * T))


def _smear(x, sigma, shape):
    g = torch.exp(-(x / sigma) ** 2) / (math.sqrt(math.pi) * sigma) if shape == "gauss" else \
        (0.5 * sigma) / (math.pi * (x * x + 0.25 * sigma * sigma))
    return torch.where(x.abs() < 2.0 * sigma, g, 0.0)


def _step2(m, mesh):
    b = TWO_PI * np.linalg.inv(m.lattice).T / np.array(mesh, float)[:, None]
    return float(np.sum(b * b) / 3.0)


def _exact_gamma(case, m, omega, evec, vel, q_list, temps):
    """Gamma [T, q in q_list, n] from the definition, dense over partners, on the GPU."""
    mesh = _mesh(case)
    pts = _points(mesh)
    N, nq, n, nb = np.array(mesh), len(pts), 3 * m.n_basis, m.n_basis
    dof = np.repeat(m.mass, 3)
    jd, kd = m.fc3_j % n, m.fc3_k % n
    jr, kr = m.fc3_j // n, m.fc3_k // n
    coef = m.fc3_val / np.sqrt(dof[m.fc3_i] * dof[jd] * dof[kd])
    # V = sum over (jr, kr, jd, kd); the phases of q1 and q2 = -q - q1 depend on (jr, kr) alone
    reps, r_of = np.unique(jr.astype(np.int64) * len(m.rep) + kr, return_inverse=True)
    A = torch.zeros(len(reps), n, n, n, dtype=torch.float64)  # [replica pair, i, j, k]
    A.view(-1).index_add_(0, torch.from_numpy(((r_of.astype(np.int64) * n + m.fc3_i) * n + jd) * n + kd),
                          torch.from_numpy(coef))
    A = A.cuda().to(torch.complex128)
    rj, rk = m.rep[reps // len(m.rep)], m.rep[reps % len(m.rep)]
    turn = lambda p, r: ((p[:, None, :] * r[None]) % N / N).sum(-1)  # noqa: E731
    ph1 = torch.polar(torch.ones(nq, len(reps), dtype=torch.float64),
                      -TWO_PI * torch.from_numpy(turn(pts, rj))).cuda()
    ph2 = torch.polar(torch.ones(nq, len(reps), dtype=torch.float64),
                      -TWO_PI * torch.from_numpy(turn(pts, rk))).cuda()
    w, e, v = _cuda(omega), _cuda(evec), _cuda(vel)
    eT = e.transpose(1, 2).contiguous()
    ok = w / TWO_PI >= NU_MIN
    wp = torch.where(ok, w, 1.0)
    h2, floor, fixed = _step2(m, mesh), TWO_PI * FLOOR, TWO_PI * SIGMA
    occ = [torch.where(ok, _bose(wp, T), 0.0) for T in temps]
    out = torch.zeros(len(temps), len(q_list), n, dtype=torch.float64, device="cuda")
    pre = math.pi * HBAR * UNIT ** 3 / 8.0 / nq
    for at, q in enumerate(q_list):
        p2 = (-pts[q][None] - pts) % N
        q2 = torch.from_numpy((p2[:, 0] * N[1] + p2[:, 1]) * N[2] + p2[:, 2]).cuda()
        w2 = w[q2]
        xs = w[:, :, None] - w2[:, None, :]           # w1 - w2
        xd = w[:, :, None] + w2[:, None, :]           # w1 + w2
        if case["adaptive"]:
            v1, v2 = v[:, :, None, :], v[q2][:, None, :, :]
            sp = ((v1 + v2).square().sum(-1) * (h2 / 12.0)).sqrt().clamp_min(floor)
            sm = ((v2 - v1).square().sum(-1) * (h2 / 12.0)).sqrt().clamp_min(floor)
        else:
            sp = sm = torch.full_like(xs, fixed)
        pair = ok[:, :, None] & ok[q2][:, None, :]
        wq = w[q][None, :, None, None]
        near = ((wq + xs[:, None]).abs() < 2.0 * sp[:, None]) | ((wq - xd[:, None]).abs() < 2.0 * sm[:, None])
        near &= pair[:, None] & ok[q][None, :, None, None]
        i1, s, s1, s2 = near.nonzero(as_tuple=True)
        B = (ph1 * ph2[q2]) @ torch.einsum("rijk,is->rsjk", A, e[q]).reshape(len(reps), -1)
        V = torch.matmul(B.reshape(nq, n * n, n), e[q2]).reshape(nq, n, n, n)      # [q1, s, j, s2]
        V = torch.matmul(eT, V.permute(0, 2, 1, 3).reshape(nq, n, n * n)).reshape(nq, n, n, n)
        V = V[i1, s1, s, s2]
        a1, a2, a0 = w[i1, s1], w2[i1, s2], w[q][s]
        gp = _smear((a0 + a1) - a2, sp[i1, s1, s2], case["shape"])
        gm = _smear((a0 - a1) - a2, sm[i1, s1, s2], case["shape"])
        k = pre * (V.real ** 2 + V.imag ** 2) / (a0 * a1 * a2)
        for t in range(len(temps)):
            n1, n2 = occ[t][i1, s1], occ[t][q2[i1], s2]
            out[t, at].index_add_(0, s, k * ((n1 - n2) * gp + 0.5 * (n1 + n2 + 1.0) * gm))
    return out


def _exact_isotopes(case, m, omega, evec, vel):
    mesh = _mesh(case)
    w, e = _cuda(omega), _cuda(evec)
    nq, n = w.shape
    ok = w / TWO_PI >= NU_MIN
    sig = torch.full_like(w, TWO_PI * SIGMA) if not case["adaptive"] else \
        (_cuda(vel).square().sum(-1) * (_step2(m, mesh) / 12.0)).sqrt().clamp_min(TWO_PI * FLOOR)
    g = _g_factor(case)
    atoms = e.reshape(nq, m.n_basis, 3, n).permute(1, 2, 0, 3).reshape(m.n_basis, 3, nq * n)
    out = torch.zeros_like(w)
    for q in range(nq):
        eq = e[q].reshape(m.n_basis, 3, n)
        o = sum(g[i] * (eq[i].conj().T @ atoms[i]).abs() ** 2 for i in range(m.n_basis) if g[i])
        d = _smear(w[q][:, None] - w.reshape(1, -1), sig.reshape(1, -1).expand(n, -1), case["shape"])
        d = torch.where(ok.reshape(1, -1), d, 0.0)
        out[q] = torch.where(ok[q], math.pi / (2.0 * nq) * w[q] ** 2 * (d * o).sum(1), 0.0)
    return out


def _carriers(w, gamma):
    return (w / TWO_PI >= NU_MIN) & (gamma > 1e-8 * gamma.max()) & (gamma > 0)


def _exact_kappa(m, omega, vel, gamma, T):
    w, v = _cuda(omega), _cuda(vel)
    use = _carriers(w, gamma)
    x = HBAR * torch.where(use, w, 1.0) / (KB * T)
    c = torch.where(use, x * x * torch.exp(x) / torch.expm1(x) ** 2 / (2.0 * torch.where(use, gamma, 1.0)), 0.0)
    v = v.reshape(-1, 3)
    return KAPPA_UNIT / (w.shape[0] * m.volume) * ((c.reshape(-1, 1) * v).T @ v)


def _exact_glass(case, m):
    omega, E = (_cuda(x) for x in _glass_modes(m))
    n = len(omega)
    dof = torch.from_numpy(np.repeat(m.mass, 3)).cuda()
    i, j, k = (torch.from_numpy(x.astype(np.int64)).cuda() for x in (m.fc3_i, m.fc3_j, m.fc3_k))
    coef = torch.from_numpy(m.fc3_val).cuda() / (dof[i] * dof[j] * dof[k]).sqrt()
    ok = omega / TWO_PI >= NU_MIN
    wp = torch.where(ok, omega, 1.0)
    occ = torch.where(ok, _bose(wp, case["kelvin"]), 0.0)
    pair = ok[:, None] & ok[None, :]
    sigma = torch.full((), TWO_PI * SIGMA, dtype=torch.float64, device="cuda")
    ET = E.T.contiguous()
    gamma = torch.zeros_like(omega)
    for mu in ok.nonzero().flatten().tolist():
        A = torch.zeros(n * n, dtype=torch.float64, device="cuda")
        A.index_add_(0, j * n + k, coef * E[i, mu])
        V = ET @ (A.view(n, n) @ E)
        w = omega[mu]
        gp = _smear((w + omega[:, None]) - omega[None, :], sigma, case["shape"])
        gm = _smear((w - omega[:, None]) - omega[None, :], sigma, case["shape"])
        pop = (occ[:, None] - occ[None, :]) * gp + 0.5 * (occ[:, None] + occ[None, :] + 1.0) * gm
        gamma[mu] = torch.where(pair, V * V * pop / (w * wp[:, None] * wp[None, :]), 0.0).sum()
    gamma *= math.pi * HBAR * UNIT ** 3 / 8.0
    if not case["extra"]:
        return {"gamma": gamma}
    use = _carriers(omega, gamma).nonzero().flatten()
    w, g, T = omega[use], gamma[use], case["kelvin"]
    dw = w[None, :] - w[:, None]
    x = HBAR * w / (KB * T)
    cm = x * x * torch.exp(x) / torch.expm1(x) ** 2
    occ = _bose(w, T)
    close = dw.abs() / TWO_PI < 1e-4
    c = HBAR / (KB * T) * w[:, None] * w[None, :] * (occ[:, None] - occ[None, :]) / torch.where(close, 1.0, dw)
    c = torch.where(close, 0.5 * (cm[:, None] + cm[None, :]), c)
    gg = 0.5 * (g[:, None] + g[None, :])
    tau = gg / (2.0 * (dw * dw + gg * gg))
    D = m.fc2[:, 0, :] / np.sqrt(np.outer(dof.cpu().numpy(), dof.cpu().numpy())) * UNIT
    sep = m.frac[None] - m.frac[:, None]
    sep = np.repeat(np.repeat((sep - np.round(sep)) @ m.lattice, 3, axis=0), 3, axis=1)
    Eu = E[:, use].contiguous()
    norm = 1.0 / (2.0 * torch.sqrt(w[:, None] * w[None, :]))
    G = [Eu.T.contiguous() @ (_cuda(D * sep[:, :, a]) @ Eu) * norm for a in range(3)]
    kappa = torch.stack([torch.stack([(c * tau * G[a] * G[b]).sum() for b in range(3)]) for a in range(3)])
    diff = torch.zeros_like(omega)
    diff[use] = (tau * (G[0] ** 2 + G[1] ** 2 + G[2] ** 2)).sum(1) / 3.0
    return {"gamma": gamma, "kappa": KAPPA_UNIT / m.volume * kappa, "diffusivity": diff}


def _stars(m, mesh):
    """Smallest mesh index in the star of each q under the 48 cubic operations."""
    pts, N = _points(mesh), np.array(mesh)
    B = TWO_PI * np.linalg.inv(m.lattice).T
    ir = np.arange(len(pts))
    for perm in itertools.permutations(range(3)):
        for sign in itertools.product((1.0, -1.0), repeat=3):
            k = ((pts / N) @ B)[:, perm] * np.array(sign) @ np.linalg.inv(B) * N
            k = np.rint(k).astype(int) % N
            ir = np.minimum(ir, (k[:, 0] * N[1] + k[:, 1]) * N[2] + k[:, 2])
    return ir


def exact(case, seed):
    """What run() gives for these inputs in plain 64-bit torch and numpy.  Linewidths depend on
    the basis inside degenerate multiplets, so a whole run pins its frequencies alone, and the
    inversion, which starts from the library's phonons, has no value here."""
    kind = case["kind"]
    if kind == "bte":
        return None
    m = _build(case, seed)
    if kind == "glass":
        return _exact_glass(case, m)
    mesh = _mesh(case)
    omega, evec, vel = _phonons(m, mesh)
    if kind == "run":
        return {"omega": omega, "evec": None, "vel": None, "gamma": None, "kappa": None}
    nq = len(omega)
    if kind == "wedge":
        ir = _stars(m, mesh)
        reps = np.unique(ir)
        g = _exact_gamma(case, m, omega, evec, vel, reps, [case["kelvin"]])[0].cpu().numpy()
        for at, q in enumerate(reps):  # the mean over each run of neighbours closer than 1e-4 THz
            cuts = np.flatnonzero(np.diff(omega[q] / TWO_PI) >= 1e-4) + 1
            for part in np.split(np.arange(omega.shape[1]), cuts):
                g[at, part] = g[at, part].mean()
        return {"gamma": g[np.searchsorted(reps, ir)]}
    if kind == "sweep":
        return {"gamma": _exact_gamma(case, m, omega, evec, vel, range(nq), SWEEP_T)}
    gamma = _exact_gamma(case, m, omega, evec, vel, range(nq), [case["kelvin"]])[0]
    if case["extra"]:
        gamma = gamma + _exact_isotopes(case, m, omega, evec, vel)
    return {"gamma": gamma, "kappa": _exact_kappa(m, omega, vel, gamma, case["kelvin"])}
