"""Performance cases: the work a user of the hole k.p library has it do.

Every case is one call of a public entry point with the inputs such a program
holds at that point (fields, orbitals, a charge), made on the GPU from a seed:

  solve    lowest eigenpairs of one Hamiltonian, or of a batch (a gate sweep)
  apply    H X on a block of spinors (residuals, expectation values)
  sp       the self-consistent Schroedinger-Poisson loop
  poisson  one electrostatic solve on the device box
  ci       the two-hole configuration interaction on spin-free orbitals
  gmat     g-matrices of the bonding and antibonding doublets
  hf       Hellmann-Feynman gradient with respect to the gate voltages
  density  hole density of occupied states
  soi      spin-orbit matrix of spin-free orbitals

Solves return their eigenvalues: eigenvectors carry a free phase, and near
degeneracies a free rotation, and residual norms are rounding noise below the
tolerance.  Tolerances of the eigensolves are those at which the eigenvalues
(quadratic in the residual) are converged beyond nine digits.

exact() restates each calculation in plain torch in 64 bits.
"""

import itertools
import math

import numpy as np
import torch

import paper_2607_08447_amd as hkp

# unit constants (eV, nm, T) and the default silicon parameters
E0 = 0.03809982116            # hbar^2 / (2 m0)
MU_B = 5.788381806e-5
E_HBAR = 1.519267448e-3       # e / hbar
E_EPS0 = 1.602176634e-19 / 8.8541878128e-12 * 1e9
G1, G2, G3, DSO, KAPPA = 4.285, 0.339, 1.446, 0.044, -0.42
AV, BB, DD = 2.46, -2.35, -5.32

F64, C128 = torch.float64, torch.complex128


# ---------------------------------------------------------------------------
# cases
# ---------------------------------------------------------------------------
def _solve(nx, ny, nz, nev, nb=0, precision="mixed", batch=0, strain=True, b=(0.5, 0.0, 0.0),
           product=False, spin_free=False, graph=False, h=0.4, tol=0.0):
    return dict(kind="solve", nx=nx, ny=ny, nz=nz, h=h, nev=nev, nb=nb, precision=precision,
                batch=batch, strain=strain, bx=b[0], by=b[1], bz=b[2], product=product,
                spin_free=spin_free, graph=graph,
                tol=tol or (1e-7 if precision == "mixed" else 1e-8))


def _box(kind, nx, ny, nz, px, py, pz, **kw):
    """A Schroedinger grid inside a Poisson box, as far from the bottom contact as a third
    of the free height."""
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, px=px, py=py, pz=pz, ox=(px - nx) // 2,
                oy=(py - ny) // 2, oz=(pz - nz) * 2 // 5, h=0.4, **kw)


def listed():
    return [
        # a quick look at a small dot, and what a test or a notebook runs: launch bound
        dict(_solve(10, 8, 8, 8, 16, "fp64", strain=False, b=(0.0, 0.0, 0.0), h=0.5, tol=1e-9),
             name="solve_dot_10x8x8_fp64"),
        # one quantum dot under five gates, a field along the channel
        dict(_solve(128, 40, 40, 16), name="solve_fin_128x40x40_mixed"),
        # the double dot of the benchmark, 32 states: the largest solve
        dict(_solve(256, 48, 48, 32, 40), name="solve_dqd_256x48x48_mixed"),
        # a detuning sweep in one recorded graph, the filter in product form
        dict(_solve(96, 32, 32, 8, batch=8, product=True, graph=True),
             name="sweep_8x96x32x32_mixed"),
        # the orbital basis of a configuration interaction (odd cross-section)
        dict(_solve(128, 37, 37, 8, 0, "fp64", b=(0.0, 0.0, 0.0), spin_free=True, tol=1e-9),
             name="orbitals_128x37x37_fp64"),
        # the loop on a short fin: many small solves after each other
        _box("sp", 24, 8, 8, 30, 14, 14, nev=8, n_holes=2.0, T=4.0, anneal=15.0,
             name="sp_loop_24x8x8"),
        # H X on a block of states of the double dot, field tilted out of the plane
        dict(kind="apply", nx=256, ny=48, nz=48, h=0.4, nvec=8, strain=True, bx=0.3, by=0.2,
             bz=0.6, name="apply_256x48x48_8"),
        # the same on a ragged grid, one doublet, no strain and field
        dict(kind="apply", nx=75, ny=31, nz=29, h=0.4, nvec=2, strain=False, bx=0.0, by=0.0,
             bz=0.0, name="apply_75x31x29_2"),
        # electrostatics of the whole device (1.5 million nodes) from its charge
        _box("poisson", 256, 48, 48, 272, 64, 88, name="poisson_272x64x88"),
        # two holes in the lowest four orbitals
        _box("ci", 256, 48, 48, 272, 64, 88, M=4, name="ci_256x48x48_4"),
        # g-tensors of the double dot
        dict(kind="gmat", nx=256, ny=48, nz=48, h=0.4, strain=True, name="gmat_256x48x48"),
        # gradient of eight levels with respect to five gate voltages
        dict(kind="hf", nx=192, ny=40, nz=40, h=0.4, nev=8, G=5, name="hf_192x40x40_8"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "apply", "apply", "poisson", "poisson", "ci",
                       "gmat", "hf", "density", "soi", "sp"])
    nx, ny, nz = _log(rng, 12, 256), rng.randint(8, 48), rng.randint(8, 48)
    if rng.random() < 0.4:
        nx = max(64, nx // 64 * 64)
    b = rng.choice([(0.0, 0.0, 0.0), (0.5, 0.0, 0.0), (0.3, 0.2, 0.6),
                    (round(rng.uniform(0.1, 2.0), 2), 0.0, 0.0)])
    strain = rng.random() < 0.7
    if kind == "solve":
        prec = rng.choice(["mixed", "mixed", "fp64"])
        spin_free = prec == "fp64" and rng.random() < 0.4
        batch = rng.choice([0, 0, 0, 4, 6])
        if batch:
            nx, ny, nz = min(nx, 128), min(ny, 28), min(nz, 28)
        elif prec == "fp64":
            nx = min(nx, 128)
        return _solve(nx, ny, nz, rng.choice([2, 4, 8, 13, 16]), precision=prec, batch=batch,
                      strain=strain, b=(0.0, 0.0, 0.0) if spin_free else b,
                      product=rng.random() < 0.4, spin_free=spin_free, graph=batch > 0)
    if kind == "apply":
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, h=0.4, nvec=_log(rng, 1, 16), strain=strain,
                    bx=b[0], by=b[1], bz=b[2])
    if kind in ("poisson", "ci"):
        kw = {} if kind == "poisson" else {"M": rng.randint(1, 4)}
        return _box(kind, nx, ny, nz, nx + rng.randint(2, 16), ny + rng.randint(2, 16),
                    nz + rng.randint(6, 40), **kw)
    if kind == "sp":
        n = (rng.randint(14, 40), rng.randint(6, 10), rng.randint(6, 10))
        return _box(kind, *n, n[0] + rng.randint(4, 8), n[1] + rng.randint(4, 8),
                    n[2] + rng.randint(6, 10), nev=8, n_holes=2.0, T=4.0, anneal=15.0)
    if kind == "gmat":
        return dict(kind=kind, nx=max(nx, 32), ny=ny, nz=nz, h=0.4, strain=strain)
    if kind == "soi":
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, h=0.4, M=rng.randint(1, 16))
    if kind == "hf":
        return dict(kind=kind, nx=nx, ny=ny, nz=nz, h=0.4, nev=_log(rng, 1, 32),
                    G=rng.randint(1, 9))
    return dict(kind=kind, nx=nx, ny=ny, nz=nz, h=0.4, nev=_log(rng, 1, 32))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 7919 + 17)
    return g


def _uni(g, lo, hi, n=1):
    return (lo + (hi - lo) * torch.rand(n, generator=g, device="cuda", dtype=F64)).tolist()


def _smooth(g, shape, sigma, cells=10):
    """Zero-mean random field of standard deviation sigma, smooth over about `cells`."""
    low = [max(2, -(-n // cells) + 2) for n in shape]
    w = torch.randn([1, 1] + low, generator=g, device="cuda", dtype=F64)
    s = torch.nn.functional.interpolate(w, size=list(shape), mode="trilinear",
                                        align_corners=True)[0, 0]
    s = s - s.mean()
    return s * (sigma / s.std())


def _axes(c):
    return [(torch.arange(n, device="cuda", dtype=F64) - (n - 1) / 2.0) * c["h"]
            for n in (c["nx"], c["ny"], c["nz"])]


def _fin(c):
    """The 4.5 eV oxide step outside a 10 x 20 nm cross-section."""
    _, y, z = _axes(c)
    out = (y.abs() > 5.0)[:, None] | (z.abs() > 10.0)[None, :]
    return torch.where(out, 4.5, 0.0).to(F64).expand(c["nx"], -1, -1).contiguous()


def _gate(x, at, fwhm=8.0):
    s = fwhm / (2.0 * math.sqrt(2.0 * math.log(2.0)))
    return torch.exp(-0.5 * ((x - at) / s) ** 2)


def _potential(c, g, barrier=None):
    """The fin with two plunger gates, a barrier between them and a little disorder."""
    x = _axes(c)[0]
    sep = min(15.0, 0.25 * c["nx"] * c["h"])
    pl, pr, br = _uni(g, -0.045, -0.035, 2) + _uni(g, 0.025, 0.035)
    br = br if barrier is None else barrier
    v = pl * _gate(x, -sep) + pr * _gate(x, sep) + br * _gate(x, 0.0)
    return _fin(c) + v[:, None, None] + _smooth(g, (c["nx"], c["ny"], c["nz"]), 1e-3)


def _dot(c, g):
    """A soft harmonic dot (level spacing 2 meV) with a little disorder."""
    x, y, z = _axes(c)
    r2 = (x ** 2)[:, None, None] + (y ** 2)[:, None] + z ** 2
    return 0.002 ** 2 * r2 / (4.0 * G1 * E0) + _smooth(g, (c["nx"], c["ny"], c["nz"]), 5e-4, 3)


def _strain(c, g):
    """Compressive strain along z with a smooth perturbation."""
    s = torch.stack([_smooth(g, (c["nx"], c["ny"], c["nz"]), 1e-4) for _ in range(6)], dim=-1)
    s[..., 2] -= 0.003
    return s.contiguous()


def _fields(c, g):
    V = _dot(c, g) if c["nx"] * c["ny"] * c["nz"] < 1000 else _potential(c, g)
    return V, (_strain(c, g) if c.get("strain") else None)


def _envelopes(c, g, n):
    """n real smooth envelopes under the gates, vanishing at the walls."""
    x, y, z = _axes(c)
    cy = torch.cos(math.pi * y / (c["h"] * (c["ny"] + 1)))
    cz = torch.cos(math.pi * z / (c["h"] * (c["nz"] + 1)))
    wx = torch.cos(math.pi * x / (c["h"] * (c["nx"] + 1)))
    sep = min(15.0, 0.25 * c["nx"] * c["h"])
    out = []
    for k in range(n):
        at, w = _uni(g, -1.2 * sep, 1.2 * sep)[0], _uni(g, 0.25 * sep, 0.6 * sep)[0]
        e = (_gate(x, at, 2.0 * w + 2.0) * wx)[:, None, None] * cy[:, None] * cz
        out.append(e * (1.0 + 0.2 * _smooth(g, (c["nx"], c["ny"], c["nz"]), 1.0)))
    return torch.stack(out)


def _block(c, g, n, comp):
    """n orthonormal smooth states [n, nx, ny, nz, comp], generic complex components."""
    e = _envelopes(c, g, n * 2)
    w = torch.randn((n, 2, comp), generator=g, device="cuda", dtype=C128)
    X = torch.stack([e[2 * k, ..., None] * w[k, 0] + e[2 * k + 1, ..., None] * w[k, 1]
                     for k in range(n)])
    A = X.reshape(n, -1)
    for _ in range(2):
        L = torch.linalg.cholesky((A.conj() @ A.T).cpu())
        A = torch.linalg.solve_triangular(L.conj(), torch.eye(n, dtype=C128),
                                          upper=False).cuda() @ A
    return A.reshape(X.shape).contiguous()


# time reversal on |J m_j>: T |j, m> = (-1)^(j - m) K |j, -m>
_TJ = ((3, 1.0), (2, -1.0), (1, 1.0), (0, -1.0), (5, 1.0), (4, -1.0))


def _doublets(c, g):
    """Bonding and antibonding Kramers doublets of a double dot [4, nx, ny, nz, 6]."""
    x = _axes(c)[0]
    sep = min(15.0, 0.25 * c["nx"] * c["h"])
    base = _envelopes(c, g, 2)
    prof = [(_gate(x, -sep) + 0.9 * _gate(x, sep)), (_gate(x, -sep) - 1.1 * _gate(x, sep))]
    w = torch.tensor([0.2, 1.0, 0.1, 0.3, 0.25, 0.1], device="cuda", dtype=C128)
    w = w * torch.exp(2j * math.pi * torch.rand(6, generator=g, device="cuda", dtype=F64))

    def flip(u):
        v = torch.empty_like(u)
        for m, (to, s) in enumerate(_TJ):
            v[..., to] = s * u[..., m].conj()
        return v

    states = []
    for k in range(2):
        u = (prof[k][:, None, None] * base[k].abs())[..., None] * w
        u = u + 0.1 * torch.roll(w, 1) * (base[1 - k] * prof[k][:, None, None])[..., None]
        for s in states:
            u = u - s * (s.conj() * u).sum()
        u = u / u.abs().square().sum().sqrt()
        states += [u, flip(u)]
    return torch.stack(states).contiguous()


def _electrostatics(c, g):
    """eps_r, electrodes and their potentials: the bottom face grounded, gate strips on top."""
    p = (c["px"], c["py"], c["pz"])
    eps = torch.full(p, 3.9, device="cuda", dtype=F64)
    ins = (slice(c["ox"], c["ox"] + c["nx"]), slice(c["oy"], c["oy"] + c["ny"]),
           slice(c["oz"], c["oz"] + c["nz"]))
    eps[ins] = torch.where(_fin(c) == 0.0, 11.7, 3.9).to(F64)
    fixed = torch.zeros(p, device="cuda", dtype=torch.uint8)
    phi = torch.zeros(p, device="cuda", dtype=F64)
    fixed[:, :, 0] = 1
    x = (torch.arange(p[0], device="cuda", dtype=F64) - (p[0] - 1) / 2.0) * c["h"]
    volts = _uni(g, -0.32, -0.28, 2) + _uni(g, -0.06, -0.04)
    strips = ((-15.0, volts[0]), (15.0, volts[1]), (0.0, volts[2]))
    if c["nx"] * c["h"] < 40.0:          # a short fin: one plunger
        strips = ((0.0, volts[0]),)
    for at, v in strips:
        on = (x - at).abs() <= 5.0
        fixed[on, :, -1] = 1
        phi[on, :, -1] = v
    return eps, fixed, phi, ins


def prepare(case, seed):
    c, g = case, _gen(seed)
    k = c["kind"]
    s = {"case": c}
    if k == "solve":
        if c["batch"]:
            bars = [0.020 + 0.040 * i / c["batch"] for i in range(c["batch"])]
            s["V"] = torch.stack([_potential(c, g, b) for b in bars]).contiguous()
            s["strain"] = _strain(c, g) if c["strain"] else None
        else:
            s["V"], s["strain"] = _fields(c, g)
    elif k == "apply":
        s["V"], s["strain"] = _fields(c, g)
        s["X"] = _block(c, g, c["nvec"], 6)
    elif k in ("poisson", "ci", "sp"):
        s["eps"], s["fixed"], s["phi"], ins = _electrostatics(c, g)
        if k == "poisson":
            rho = torch.zeros_like(s["eps"])
            e = _envelopes(c, g, 2).square()
            rho[ins] = (e / e.sum((1, 2, 3), keepdim=True)).sum(0) / c["h"] ** 3
            s["rho"] = rho + 1e-4 * _smooth(g, rho.shape, 1.0)
        elif k == "ci":
            s["orb"] = _block(c, g, c["M"], 3)
            s["E"] = torch.tensor(sorted(_uni(g, 0.02, 0.06, c["M"])), device="cuda", dtype=F64)
        else:
            s["V"] = _fin(c)
    elif k == "gmat":
        s["V"], s["strain"] = _potential(c, g), (_strain(c, g) if c["strain"] else None)
        s["psi"] = _doublets(c, g)
    elif k == "soi":
        s["orb"] = _block(c, g, c["M"], 3)
        s["E"] = torch.tensor(sorted(_uni(g, 0.02, 0.06, c["M"])), device="cuda", dtype=F64)
    else:
        s["psi"] = _block(c, g, c["nev"], 6)
        if k == "hf":
            x = _axes(c)[0]
            at = torch.linspace(-30.0, 30.0, c["G"]).tolist()
            al = _uni(g, 0.05, 0.3, c["G"])
            s["L"] = torch.stack([(a * _gate(x, t))[:, None, None].expand(-1, c["ny"], c["nz"])
                                  for a, t in zip(al, at)]).contiguous()
            s["w"] = torch.tensor(_uni(g, 0.1, 1.0, c["nev"]), device="cuda", dtype=F64)
        else:
            s["f"] = torch.tensor(sorted(_uni(g, 0.0, 1.0, c["nev"]), reverse=True),
                                  device="cuda", dtype=F64)
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(s):
    c = s["case"]
    k = c["kind"]
    if k == "solve":
        kw = dict(strain=s["strain"], B=(c["bx"], c["by"], c["bz"]), nb=c["nb"], tol=c["tol"],
                  precision=c["precision"], graph=c["graph"], return_psi=True,
                  spin_free=c["spin_free"], cheb_product=c["product"])
        call = hkp.solve_batch if c["batch"] else hkp.solve
        return call(s["V"], c["h"], c["nev"], **kw).E
    if k == "apply":
        return hkp.apply(s["V"], c["h"], s["X"], strain=s["strain"],
                         B=(c["bx"], c["by"], c["bz"]))
    if k == "poisson":
        return hkp.poisson(s["eps"], s["fixed"], s["phi"], s["rho"], c["h"])[0]
    if k == "sp":
        r = hkp.sp_solve(s["V"], c["h"], c["nev"], (c["px"], c["py"], c["pz"]),
                         (c["ox"], c["oy"], c["oz"]), s["eps"], s["fixed"], s["phi"],
                         c["n_holes"], c["T"], tol=1e-11, tol_V=1e-10, anneal_T=c["anneal"],
                         graph=True)
        return {"phi": r.phi, "E": r.E}
    if k == "ci":
        r = hkp.ci_solve(s["orb"], s["E"], c["h"], (c["px"], c["py"], c["pz"]),
                         (c["ox"], c["oy"], c["oz"]), s["eps"], s["fixed"], return_matrix=True,
                         return_coulomb=True)
        return {"E": r.E, "H": r.H, "coulomb": r.coulomb}
    if k == "gmat":
        # the left and right doublets' own bases are free: their symmetric tensors are not
        r = hkp.g_matrices(s["psi"], s["V"], c["h"], s["strain"])
        return {"g": r.g[:2], "g_sym": r.g_sym, "centre_x": r.centre[:, 0], "E": r.E,
                "delta": r.delta, "d": r.d}
    if k == "hf":
        return hkp.hf_grad(s["psi"], s["w"], s["L"])
    if k == "density":
        return hkp.hole_density(s["psi"], s["f"], c["h"])
    return hkp.soi_matrix(s["orb"], E=s["E"])


def work(case):
    """Inputs read once and outputs written once (for an iteration: of the whole call)."""
    c, k = case, case["kind"]
    n = c["nx"] * c["ny"] * c["nz"]
    if k == "solve":
        m = max(1, c["batch"])
        comp = 3 if c["spin_free"] else 6
        return {"bytes": 8.0 * n * (m + 6 * c["strain"]) + 16.0 * comp * n * c["nev"] * m}
    if k == "apply":
        return {"bytes": 8.0 * n * (1 + 6 * c["strain"]) + 2 * 96.0 * n * c["nvec"]}
    if k == "poisson":
        return {"bytes": 33.0 * c["px"] * c["py"] * c["pz"]}
    if k == "sp":
        p = c["px"] * c["py"] * c["pz"]
        return {"bytes": 25.0 * p + 16.0 * n + 96.0 * n * c["nev"]}
    if k == "ci":
        return {"bytes": 9.0 * c["px"] * c["py"] * c["pz"] + 48.0 * n * c["M"]}
    if k == "gmat":
        return {"bytes": 8.0 * n * (1 + 6 * c["strain"]) + 4 * 96.0 * n}
    if k == "hf":
        return {"bytes": 96.0 * n * c["nev"] + 8.0 * n * c["G"]}
    if k == "density":
        return {"bytes": 96.0 * n * c["nev"] + 8.0 * n}
    return {"bytes": 48.0 * n * c["M"]}


# ---------------------------------------------------------------------------
# the same in plain torch, 64 bits
# ---------------------------------------------------------------------------
def _consts():
    r2, r3 = math.sqrt(2.0), math.sqrt(3.0)
    U = torch.tensor([[1j * r3, r3, 0, 0, 0, 0], [0, 0, -2j, 1j, 1, 0], [-1j, 1, 0, 0, 0, -2j],
                      [0, 0, 0, -1j * r3, r3, 0], [0, 0, -1j * r2, -1j * r2, -r2, 0],
                      [-1j * r2, r2, 0, 0, 0, 1j * r2]], dtype=C128) / math.sqrt(6.0)
    sig = torch.tensor([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=C128)
    eps = torch.zeros((3, 3, 3), dtype=C128)
    for a, b, d in ((0, 1, 2), (1, 2, 0), (2, 0, 1)):
        eps[a, b, d], eps[b, a, d] = 1.0, -1.0
    return U, sig, -1j * eps


def _shift(u, ax, up):
    """u(r + e_ax) (up) or u(r - e_ax) on [n, x, y, z, ...], zero past the wall."""
    out = torch.zeros_like(u)
    n = u.shape[ax + 1]
    if n > 1:
        a, b = (0, 1) if up else (1, 0)
        out.narrow(ax + 1, a, n - 1).copy_(u.narrow(ax + 1, b, n - 1))
    return out


def _phases(c, B, ax):
    """Link phase exp(i (e/hbar) h A_ax) at the middle of the link r -> r + e_ax."""
    r = _axes(c)
    r[ax] = r[ax] + 0.5 * c["h"]
    X, Y, Z = r[0][:, None, None], r[1][:, None], r[2]
    one = torch.ones((c["nx"], c["ny"], c["nz"]), device="cuda", dtype=F64)
    A = (0.5 * (B[1] * Z - B[2] * Y), 0.5 * (B[2] * X - B[0] * Z), 0.5 * (B[0] * Y - B[1] * X))
    return torch.polar(one, E_HBAR * c["h"] * A[ax] * one)


def _h_ls(c, V, strain, B, so, u):
    """H u for u [n, x, y, z, m] in the |L S> basis (m = 6), or orbitals (m = 3, no field)."""
    h, m = c["h"], u.shape[-1]
    ph = [None if not any(B) else _phases(c, B, a)[..., None] for a in range(3)]

    def fwd(v, a):
        s = _shift(v, a, True)
        return s if ph[a] is None else ph[a] * s

    def bwd(v, a):
        return _shift(v if ph[a] is None else ph[a].conj() * v, a, False)

    L, M, N = G1 + 4 * G2, G1 - 2 * G2, 6 * G3
    u = u.reshape(u.shape[:-1] + (m // 3, 3))
    out = torch.zeros_like(u)
    for s in range(m // 3):
        w = u[..., s, :]
        o = torch.zeros_like(w)
        first = []
        for a in range(3):
            f, b = fwd(w, a), bwd(w, a)
            cf = torch.full((3,), M, device="cuda", dtype=F64)
            cf[a] = L
            o += (E0 / h ** 2) * cf * (2 * w - f - b)
            first.append(-1j * (f - b) / (2 * h))
        for a in range(3):
            for b in range(3):
                if a != b:      # symmetrised k_a k_b on component b into component a
                    t = 0.0
                    for p, q in ((a, b), (b, a)):
                        d = first[q][..., b:b + 1]
                        t = t - 0.5j * (fwd(d, p) - bwd(d, p)) / (2 * h)
                    o[..., a:a + 1] += E0 * N * t
        out[..., s, :] = o
    del first, o
    if strain is not None:
        l, mm, nn = -(AV + 2 * BB), -(AV - BB), -math.sqrt(3.0) * DD
        tr = strain[..., 0] + strain[..., 1] + strain[..., 2]
        D = torch.zeros(strain.shape[:-1] + (3, 3), device="cuda", dtype=F64)
        for i in range(3):
            D[..., i, i] = l * strain[..., i] + mm * (tr - strain[..., i])
        for i, j, v in ((1, 2, 3), (0, 2, 4), (0, 1, 5)):
            D[..., i, j] = D[..., j, i] = nn * strain[..., v]
        for i in range(3):
            for j in range(3):
                out[..., i] += D[..., i, j][..., None] * u[..., j]
    out += V[..., None, None] * u
    out = out.reshape(out.shape[:-2] + (m,))
    if m == 6:
        on = (_so_matrix() if so else torch.zeros((6, 6), dtype=C128)) + _zeeman(B)
        out += u.reshape(out.shape) @ on.T.cuda()
    return out


def _so_matrix():
    _, sig, lo = _consts()
    return DSO / 3.0 * (torch.eye(6, dtype=C128) - sum(torch.kron(sig[a], lo[a]) for a in range(3)))


def _zeeman(B):
    _, sig, lo = _consts()
    i2, i3 = torch.eye(2, dtype=C128), torch.eye(3, dtype=C128)
    return MU_B * sum(B[a] * ((3 * KAPPA - 1) * torch.kron(i2, lo[a]) + torch.kron(sig[a], i3))
                      for a in range(3))


def _exact_solve(c, s):
    m = 3 if c["spin_free"] else 6
    n = c["nx"] * c["ny"] * c["nz"] * m
    if n > 4000:          # a dense diagonalisation beyond this takes too long
        return None
    E = []
    for V in (s["V"] if c["batch"] else [s["V"]]):
        eye = torch.eye(n, device="cuda", dtype=C128).reshape(n, c["nx"], c["ny"], c["nz"], m)
        H = torch.cat([_h_ls(c, V, s["strain"], (c["bx"], c["by"], c["bz"]), True, e)
                       for e in eye.split(256)]).reshape(n, n)
        E.append(torch.from_numpy(np.linalg.eigvalsh(H.cpu().numpy())[:c["nev"]]).cuda())
    return torch.stack(E) if c["batch"] else E[0]


def _laplace(c, eps, fixed):
    """Link coefficients of the 7-point Poisson operator on the free nodes, and its diagonal."""
    cs, diag = [], torch.zeros_like(eps)
    for a in range(3):
        n = eps.shape[a]
        p, q = eps.narrow(a, 0, n - 1), eps.narrow(a, 1, n - 1)
        k = 2 * p * q / (p + q) / c["h"] ** 2
        diag.narrow(a, 0, n - 1).add_(k)
        diag.narrow(a, 1, n - 1).add_(k)
        cs.append(k)
    return cs, diag, (fixed == 0).to(F64)


def _lap(op, u):
    cs, diag, _ = op
    out = diag * u
    for a, k in enumerate(cs):
        n, ax = u.shape[a + 1], a + 1
        out.narrow(ax, 0, n - 1).sub_(k * u.narrow(ax, 1, n - 1))
        out.narrow(ax, 1, n - 1).sub_(k * u.narrow(ax, 0, n - 1))
    return out


def _cg(op, b, tol=1e-15, most=4000):
    """Jacobi-preconditioned conjugate gradients for several right-hand sides at once."""
    free, inv = op[2], op[2] / op[1]
    b = b * free
    dot = lambda x, y: (x * y).sum((1, 2, 3), keepdim=True)  # noqa: E731
    x, r = torch.zeros_like(b), b.clone()
    z = inv * r
    p, rz, bb = z.clone(), dot(r, z), dot(b, b)
    tiny = torch.finfo(F64).tiny
    for it in range(most):
        q = _lap(op, p) * free
        al = rz / (dot(p, q) + tiny)
        x += al * p
        r -= al * q
        if it % 20 == 0 and bool((dot(r, r) <= tol ** 2 * bb).all()):
            break
        z = inv * r
        rz2 = dot(r, z)
        p = z + rz2 / (rz + tiny) * p
        rz = rz2
    return x


def _refined(op, b):
    """Two rounds: the second on the residual of the first."""
    x = _cg(op, b)
    return x + _cg(op, b * op[2] - _lap(op, x) * op[2], 1e-6)


def _soi(orb, E):
    M = orb.shape[0]
    p = orb.reshape(M, -1, 3)
    O = torch.stack([torch.stack([p[:, :, b].conj() @ p[:, :, d].T for d in range(3)])
                     for b in range(3)]).cpu()                       # [b, d, i, j]
    hso = _so_matrix().reshape(2, 3, 2, 3)
    out = torch.zeros((M, 2, M, 2), dtype=C128)
    for s, b, t, d in itertools.product(range(2), range(3), range(2), range(3)):
        out[:, s, :, t] += O[b, d] * hso[s, b, t, d]
    out = out.reshape(2 * M, 2 * M)
    return out + torch.kron(torch.diag(E.cpu().to(C128)), torch.eye(2, dtype=C128))


def _exact_ci(c, s):
    M, h3 = c["M"], c["h"] ** 3
    op = _laplace(c, s["eps"], s["fixed"])
    orb = s["orb"]
    ins = (slice(c["ox"], c["ox"] + c["nx"]), slice(c["oy"], c["oy"] + c["ny"]),
           slice(c["oz"], c["oz"] + c["nz"]))
    rho = {(i, k): (orb[i].conj() * orb[k]).sum(-1) / h3 for i in range(M) for k in range(M)}
    C = torch.zeros((M, M, M, M), dtype=C128)
    for j in range(M):
        for l in range(j, M):
            b = torch.zeros((2,) + tuple(s["eps"].shape), device="cuda", dtype=F64)
            b[(0,) + ins], b[(1,) + ins] = rho[j, l].real, rho[j, l].imag
            v = _cg(op, E_EPS0 * b, 1e-14)
            v = torch.complex(v[0], v[1])[ins]
            for i in range(M):
                for k in range(M):
                    C[i, k, j, l] = complex(h3 * (rho[i, k] * v).sum())
                    C[i, k, l, j] = complex(h3 * (rho[i, k] * v.conj()).sum())
    hs = _soi(orb, s["E"])
    dets = list(itertools.combinations(range(2 * M), 2))
    H = np.zeros((len(dets),) * 2, dtype=complex)
    hs_, C_ = hs.numpy(), C.numpy()

    def two(u, v, w, x):
        same = (u & 1) == (w & 1) and (v & 1) == (x & 1)
        return C_[u >> 1, w >> 1, v >> 1, x >> 1] if same else 0.0

    for a, (u, v) in enumerate(dets):
        for b, (w, x) in enumerate(dets):
            H[a, b] = (hs_[u, w] * (v == x) + hs_[v, x] * (u == w) - hs_[u, x] * (v == w)
                       - hs_[v, w] * (u == x) + two(u, v, w, x) - two(u, v, x, w))
    return {"E": np.linalg.eigvalsh(H), "H": H, "coulomb": C}


def _exact_gmat(c, s):
    U, sig, _ = _consts()
    u = s["psi"] @ U.conj().cuda()                      # |L S> components: U^H psi
    r = [a.reshape([-1 if i == k else 1 for i in range(3)] + [1])
         for k, a in enumerate(_axes(c))]
    H0 = [_h_ls(c, s["V"], s["strain"], (0, 0, 0), True, w) for w in
          [u] + [ra * u for ra in r]]
    ip = lambda p, q: (p.reshape(4, -1).conj() @ q.reshape(4, -1).T).cpu()  # noqa: E731
    one = ip(u, u)
    E = ip(u, H0[0]).diagonal().real
    X = [ip(u, ra * u) for ra in r]
    W = [[ip(r[p] * u, H0[q + 1]) for q in range(3)] for p in range(3)]
    A = [ip(u, H0[q + 1]) for q in range(3)]             # <psi| H0 R_q |psi>
    Hm = ip(u, H0[0])
    Z = [ip(u, u @ _zeeman([float(b == a) for a in range(3)]).T.cuda()) for b in range(3)]
    _, Cx = np.linalg.eigh((0.5 * (X[0] + X[0].conj().T)).numpy())
    Cx = torch.from_numpy(Cx)
    idn = torch.eye(4, dtype=C128)
    subs = [idn[:, :2], idn[:, 2:], Cx[:, :2], Cx[:, 2:]]
    gs, syms, cen = [], [], []
    for T in subs:
        pr = lambda m: T.conj().T @ m @ T  # noqa: E731
        r0 = [float(pr(X[a]).diagonal().real.mean()) for a in range(3)]
        cen.append(r0)
        g = np.zeros((3, 3))
        for b in range(3):
            p, q = (b + 1) % 3, (b + 2) % 3

            def w(i, j):
                return (W[i][j] - r0[i] * A[j] - r0[j] * A[i].conj().T + r0[i] * r0[j] * Hm)

            Mb = pr(Z[b] + 0.5j * E_HBAR * (w(p, q) - w(q, p)))
            for a in range(3):
                g[a, b] = float(torch.trace(sig[a] @ Mb).real) / MU_B
        w_, Q = np.linalg.eigh(g.T @ g)
        gs.append(g)
        syms.append((-1.0 if np.linalg.det(g) < 0 else 1.0) * (Q * np.sqrt(np.maximum(w_, 0))) @ Q.T)
    del one
    cen = np.array(cen)
    return {"g": np.array(gs[:2]), "g_sym": np.array(syms), "centre_x": cen[:, 0],
            "E": E.numpy(), "delta": float(0.5 * (E[2] + E[3]) - 0.5 * (E[0] + E[1])),
            "d": float(np.linalg.norm(cen[3] - cen[2]))}


def exact(case, seed):
    c, s = case, prepare(case, seed)
    k = c["kind"]
    if k == "solve":
        return _exact_solve(c, s)
    if k == "apply":
        U = _consts()[0].cuda()
        out = [_h_ls(c, s["V"], s["strain"], (c["bx"], c["by"], c["bz"]), True, x @ U.conj())
               @ U.T for x in s["X"].split(2)]
        return torch.cat(out)
    if k == "poisson":
        op = _laplace(c, s["eps"], s["fixed"])
        lift = (s["phi"] * (1 - op[2]))[None]
        b = (E_EPS0 * s["rho"])[None] - _lap(op, lift)
        return (lift + _refined(op, b))[0]
    if k == "ci":
        return _exact_ci(c, s)
    if k == "gmat":
        return _exact_gmat(c, s)
    if k == "hf":
        n = s["psi"].abs().square().sum(-1)
        return torch.stack([(s["w"][:, None, None, None] * n * L).sum() for L in s["L"]])
    if k == "density":
        n = s["psi"].abs().square().sum(-1)
        return (s["f"][:, None, None, None] * n).sum(0) / c["h"] ** 3
    if k == "soi":
        return _soi(s["orb"], s["E"])
    return None           # the loop: its fixed point has no short restatement
