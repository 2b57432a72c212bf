"""The work whose speed is measured: calls of the library's entry points at
the sizes users run them.

The listed cases stand for an excited-state calculation as the solvers and the
relaxation driver make it: the operator apply on blocks of trial vectors (the
inner loop of Davidson) from the micro system to the 72^3 supercell grid, in
FP64 and mixed precision, with the pair potentials cached, partly cached, and
replayed through HIP graphs; the U vector and the Z-vector solve; the coupling
apply beyond the Tamm-Dancoff approximation; and one whole geometry from the
ground state to the forces.  The systems follow the synthetic configurations:
cubic cells of 10 N / 24 bohr at 10 Ha (``c1``, the ``c4`` family), the 12^3
micro system, the 72^3 supercell and the 48 x 48 x 120 slab; band counts lie in
the configurations' range, kept so that a few contexts fit one device.

Inputs are drawn from the case's seed on the GPU.  Operator cases use smooth
orthonormal orbitals with made-up energies and trial vectors of standard
normals (the operator assumes no eigenpairs); the solver cases solve the ground
state of sites displaced by a few hundredths of a bohr, as a relaxation does.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2607_20728_amd import bsex

GRIDS = (12, 16, 20, 24, 30, 32, 36, 40, 45, 48, 50, 54, 60, 64, 72)
N_SITES = 8


def _case(name, kind, grid, n_val, n_pdep, n_b=1, mixed=False, tau_gb=0.0, graphs=False, cell=None,
          ecut=10.0):
    cell = cell or [10.0 * n / 24.0 for n in grid]
    c = dict(kind=kind, n1=grid[0], n2=grid[1], n3=grid[2], l1=cell[0], l2=cell[1], l3=cell[2],
             ecut=ecut, n_val=n_val, n_pdep=n_pdep, n_b=n_b, mixed=mixed, tau_gb=tau_gb,
             graphs=graphs)
    if name:
        c["name"] = name
    return c


def listed():
    cubic = [20.2] * 3
    slab = [47.34, 40.99, 110.0]
    return [
        # the smallest call: one vector on the micro system, launches and latency
        _case("apply_micro", "apply", (12, 12, 12), 4, 8, cell=[8.0] * 3, ecut=4.0),
        # the tiny system's Davidson block (one exciton and four more vectors)
        # replayed through a HIP graph, as the batch runner does
        _case("apply_24_graph", "apply", (24, 24, 24), 16, 64, n_b=5, graphs=True),
        # a small batch member with an odd band count
        _case("apply_32", "apply", (32, 32, 32), 107, 211, n_b=5),
        # ragged grid lengths, odd bands, few vectors
        _case("apply_ragged", "apply", (36, 45, 50), 61, 150, n_b=3),
        # a throughput block on a middle grid in mixed precision
        _case("apply_48_mixed", "apply", (48, 48, 48), 180, 256, n_b=8, mixed=True),
        # a large batch member, whole tau cache streamed: the usual bound
        _case("apply_64", "apply", (64, 64, 64), 200, 320, n_b=8),
        # the supercell grid with a cache that holds half of tau: the rest is
        # rebuilt inside the call, as in its FP64 Davidson
        _case("apply_72_partial", "apply", (72, 72, 72), 256, 512, n_b=8, tau_gb=50.0, cell=cubic,
              ecut=14.2),
        # the U vector: every pair density of the exciton through W
        _case("u_64", "u", (64, 64, 64), 200, 320),
        # the same on the slab in mixed precision
        _case("u_slab_mixed", "u", (48, 48, 120), 160, 256, mixed=True, cell=slab, ecut=3.26),
        # U and the Z-vector solve on a middle batch member
        _case("zvector_40", "zvector", (40, 40, 40), 96, 200),
        # beyond the Tamm-Dancoff approximation: the coupling apply
        _case("coupling_32", "coupling", (32, 32, 32), 48, 160, n_b=2),
        # one geometry of a relaxation: ground state, tau, exciton, U, Z, forces
        _case("geometry_32", "geometry", (32, 32, 32), 33, 128),
    ]


def draw(rng):
    def log_int(a, b):
        return int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))

    while True:
        kind = rng.choices(("apply", "u", "coupling", "zvector", "geometry"), (10, 3, 2, 2, 1))[0]
        if rng.random() < 0.6:
            grid = [rng.choice(GRIDS)] * 3
        else:
            grid = [rng.choice(GRIDS) for _ in range(3)]
        nr = grid[0] * grid[1] * grid[2]
        npw = 0.1 * nr
        if nr % 2 or nr > 72 ** 3:
            continue
        nv = log_int(3, 256)
        npd = log_int(8, 512)
        if nv > npw / 4 or npd > npw / 3:
            continue
        blocks = ((nv + 7) // 8) * ((nv + 7) // 8 + 1) // 2
        mixed = kind in ("apply", "u") and rng.random() < 0.3
        nb = rng.randint(1, 16) if kind == "apply" else rng.randint(1, 2) if kind == "coupling" else 1
        tau_gb, graphs = 0.0, False
        tau = blocks * 64.0 * nr * 8
        if kind == "apply":
            if tau > (26e9 if mixed else 40e9):
                continue
            graphs = rng.random() < 0.2
            if not mixed and rng.random() < 0.2:
                tau_gb = max(0.01, rng.uniform(0.2, 0.9) * tau / 1e9)
                if (blocks - tau_gb * 1e9 / (tau / blocks)) * nr * ((nb + 7) // 8) > 2.5e7:
                    continue
        if kind == "u" and blocks * nr > 8e7:
            continue
        if kind == "coupling" and nv * nv * nr * nb > 4e8:
            continue
        if kind == "zvector" and (nr > 48 ** 3 or not 8 <= nv <= 96 or min(grid) < 24):
            continue
        if kind == "geometry" and (nr > 32 ** 3 or not 12 <= nv <= 33 or min(grid) < 24):
            continue
        return _case(None, kind, grid, nv, npd, nb, mixed, round(tau_gb, 3), graphs)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
def _sphere(case):
    """Miller indices of the half sphere and |G|^2 per basis function, in the
    documented order: G = 0, then (cos, sin) of every half-sphere vector by
    (|n|^2, n1, n2, n3)."""
    N = np.array([case["n1"], case["n2"], case["n3"]])
    L = np.array([case["l1"], case["l2"], case["l3"]])
    top = np.minimum(N, (L * math.sqrt(2 * case["ecut"]) / (2 * math.pi)).astype(int) + 1)
    ax = [np.arange(-t, t + 1) for t in top]
    m = np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)
    g2 = ((2 * math.pi * m / L) ** 2).sum(1)
    first = np.where(m[:, 0] != 0, m[:, 0], np.where(m[:, 1] != 0, m[:, 1], m[:, 2]))
    keep = (0.5 * g2 <= case["ecut"]) & (first > 0)
    m, g2 = m[keep], g2[keep]
    o = np.lexsort((m[:, 2], m[:, 1], m[:, 0], (m * m).sum(1)))
    return m[o], np.concatenate([[0.0], np.repeat(g2[o], 2)])


def _n_pw(case):
    return 1 + 2 * len(_sphere(case)[0])


def _rng(seed, salt):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 16 + salt)
    return g


def _normal(shape, seed, salt):
    return torch.randn(shape, generator=_rng(seed, salt), dtype=torch.float64, device="cuda")


def _orthonormal_rows(a):
    for _ in range(2):  # Cholesky QR, twice
        a = torch.linalg.solve_triangular(torch.linalg.cholesky(a @ a.T), a, upper=False)
    return a


def _pdep(case, npw, seed):
    """PDEP vectors [n_pw][n_pdep], orthonormal without a G = 0 component, and
    lambda_i = -0.85 exp(-i / (n_pdep / 5))."""
    n = case["n_pdep"]
    a = _normal((n, npw), seed, 1)
    a[:, 0] = 0.0
    lam = -0.85 * np.exp(-np.arange(n) / (n / 5.0))
    return _orthonormal_rows(a).T.contiguous(), lam


def _sites(case, seed, fixed):
    """Gaussian sites: positions of one fixed draw displaced by N(0, 0.03 bohr)
    (the geometries of a relaxation) or drawn afresh."""
    L = np.array([case["l1"], case["l2"], case["l3"]])
    r = np.random.Generator(np.random.PCG64(4028 if fixed else int(seed)))
    xyz = r.random((N_SITES, 3)) * L
    depth, width = r.uniform(1.0, 3.0, N_SITES), r.uniform(0.8, 1.5, N_SITES)
    if fixed:
        xyz = xyz + np.random.Generator(np.random.PCG64(int(seed))).normal(0.0, 0.03, xyz.shape)
    return xyz, depth, width


def _orbitals(case, g2, seed):
    """Smooth orthonormal orbitals and made-up ascending energies."""
    t = torch.tensor(1.0 + 0.5 * g2, device="cuda")
    n = case["n_val"]
    return _orthonormal_rows(_normal((n, len(g2)), seed, 2) / t), np.linspace(-1.0, -0.3, n)


def _system(case, seed, solve):
    _, g2 = _sphere(case)
    xyz, depth, width = _sites(case, seed, solve)
    # a relaxation keeps the dielectric basis of its first geometry
    P, lam = _pdep(case, len(g2), 0 if solve else seed)
    return dict(g2=g2, xyz=xyz, depth=depth, width=width, pdep=P, lam=lam,
                cell=[case["l1"], case["l2"], case["l3"]],
                grid=[case["n1"], case["n2"], case["n3"]])


def _init(case, s, **kw):
    return bsex.init_system(s["cell"], s["grid"], case["ecut"], s["xyz"], s["depth"], s["width"],
                            case["n_val"], s["pdep_host"], s["lam"],
                            tau_budget_bytes=int(case["tau_gb"] * 1e9),
                            precision=bsex.MIXED if case["mixed"] else bsex.FP64, **kw)


def _vectors(case, g2, seed):
    """Trial vectors [n_b][n_val][n_pw], or one smooth normalised exciton."""
    x = _normal((case["n_b"], case["n_val"], len(g2)), seed, 3)
    if case["kind"] in ("apply", "coupling"):
        return x
    x = x / torch.tensor(1.0 + 0.5 * g2, device="cuda")
    return (x / x.norm())[0].contiguous()


def prepare(case, seed):
    kind = case["kind"]
    solve = kind in ("zvector", "geometry")
    s = _system(case, seed, solve)
    s["pdep_host"] = s.pop("pdep").cpu().numpy()
    st = dict(case=case, system=s)
    if kind == "geometry":
        return st
    if solve:
        st["ctx"] = _init(case, s, n_extra=32)
    else:
        phi, eps = _orbitals(case, s["g2"], seed)
        st["ctx"] = _init(case, s, orbitals=phi.cpu().numpy(), eps=eps)
    if case["graphs"]:
        bsex.set_graphs(st["ctx"], True)
    st["X"] = _vectors(case, s["g2"], seed)
    return st


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind = case["kind"]
    if kind == "apply":
        return bsex.apply(st["ctx"], st["X"])
    if kind == "coupling":
        return bsex.apply_coupling(st["ctx"], st["X"])
    if kind == "u":
        return bsex.u_vector(st["ctx"], st["X"])
    if kind == "zvector":
        Z, _ = bsex.zvector_solve(st["ctx"], st["X"], tol=1e-6, two_level=True)
        return Z
    ctx = _init(case, st["system"], n_extra=32)
    try:
        phi, eps = bsex.get_orbitals(ctx)
        w, X, _ = bsex.davidson(ctx, 1, tol=1e-6, two_level=True)
        Z, _ = bsex.zvector_solve(ctx, X[0], tol=1e-6, two_level=True)
        dw = bsex.forces(ctx, X[0], Z, N_SITES)
        dE = bsex.ground_state_forces(ctx, N_SITES)
    finally:
        ctx.free()
    return dict(eps=eps, omega=w, X=X, Z=Z, dw=dw, dE=dE)


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    nr = case["n1"] * case["n2"] * case["n3"]
    npw, nv, nb, npd = _n_pw(case), case["n_val"], case["n_b"], case["n_pdep"]
    pairs = nv * (nv + 1) / 2
    real_fft = 2.5 * nr * math.log2(nr)                   # one real transform
    vec = nv * npw
    proj = 4.0 * nv * vec                                 # P_c of one vector set
    w_pair = nr + 2 * real_fft + 4.0 * npw * npd          # W of one pair density
    apply1 = 2 * proj + 2 * nv * real_fft + 2 * nv * nr + 4 * pairs * nr
    kind = case["kind"]
    tau = pairs * nr * (4 if case["mixed"] else 8)
    if kind == "apply":
        part = min(1.0, case["tau_gb"] * 1e9 / tau) if case["tau_gb"] else 1.0
        return dict(bytes=8.0 * vec * (2 * nb + 1) + part * tau,
                    flops=nb * apply1 + (1 - part) * pairs * w_pair)
    if kind == "coupling":
        return dict(bytes=8.0 * vec * (2 * nb + 1) + 8.0 * npw * npd,
                    flops=nb * (2 * proj + 2 * nv * real_fft + nv * nv * (w_pair + 2 * nr)))
    u = dict(bytes=8.0 * vec * 3 + 8.0 * npw * npd + tau,
             flops=apply1 + pairs * (w_pair + 4 * nr) + 2 * proj)
    if kind == "u":
        return u
    step = 2 * nv * real_fft + 2 * proj                   # one step of a solver
    if kind == "zvector":
        return dict(bytes=u["bytes"] + 8.0 * vec, flops=u["flops"] + 20 * step)
    # ground state (about 20 sweeps of degree 16), tau, Davidson (about 60
    # applies), U, Z and the forces
    gs = 20 * 17 * 2 * (nv + 32) * real_fft
    return dict(bytes=2 * tau + 8.0 * npw * npd, flops=gs + 60 * apply1 + pairs * w_pair + u["flops"]
                + 20 * step)


# ---------------------------------------------------------------------------
# the results in plain torch, FP64
# ---------------------------------------------------------------------------
class _Exact:
    def __init__(self, case, seed):
        self.case = case
        s = _system(case, seed, False)
        self.nv = case["n_val"]
        N = np.array(s["grid"])
        L = np.array(s["cell"])
        self.N = tuple(int(n) for n in N)
        self.nr, self.omega = int(N.prod()), float(L.prod())
        mill, g2 = _sphere(case)
        self.npw, self.g2 = len(g2), torch.tensor(g2, device="cuda")
        lin = lambda m: (m[:, 0] * N[1] + m[:, 1]) * N[2] + m[:, 2]  # noqa: E731
        self.ip = torch.tensor(lin(mill % N), device="cuda")
        self.im = torch.tensor(lin((-mill) % N), device="cuda")
        n = [torch.fft.fftfreq(k, 1.0 / k, dtype=torch.float64, device="cuda") for k in self.N]
        g = [2 * math.pi * a / l for a, l in zip(n, L)]
        G = torch.meshgrid(*g, indexing="ij")
        gg = G[0] ** 2 + G[1] ** 2 + G[2] ** 2
        self.vc = torch.where(gg > 0, 4 * math.pi / torch.where(gg > 0, gg, 1.0), 0.0)
        nyq = torch.zeros(self.N, dtype=torch.bool, device="cuda")
        for a in range(3):
            if self.N[a] % 2 == 0:
                nyq.index_fill_(a, torch.tensor([self.N[a] // 2], device="cuda"), True)
        VG = torch.zeros(self.N, dtype=torch.complex128, device="cuda")
        for R, d, w in zip(s["xyz"], s["depth"], s["width"]):
            ph = torch.polar(torch.ones_like(gg), -(G[0] * R[0] + G[1] * R[1] + G[2] * R[2]))
            VG += -(d / self.omega) * (2 * math.pi * w * w) ** 1.5 * torch.exp(-0.5 * w * w * gg) * ph
        VG[nyq] = 0
        self.V = (torch.fft.ifftn(VG) * self.nr).real
        vs = torch.zeros_like(self.g2)
        vs[1:] = torch.sqrt(4 * math.pi / self.g2[1:])
        lam = torch.tensor(s["lam"], device="cuda")
        self.P = s["pdep"] * vs[:, None]
        self.Pc = self.P * (lam / (1 - lam))
        self.phi, eps = _orbitals(case, g2, seed)
        self.eps = torch.tensor(eps, device="cuda")
        self.phir = self.to_grid(self.phi)
        self.X = _vectors(case, g2, seed)

    def coeffs(self, x):
        F = torch.zeros((x.shape[0], self.nr), dtype=torch.complex128, device="cuda")
        F[:, 0] = x[:, 0] / math.sqrt(self.omega)
        f = torch.complex(x[:, 1::2], -x[:, 2::2]) / math.sqrt(2 * self.omega)
        F[:, self.ip] = f
        F[:, self.im] = f.conj()
        return F.reshape((-1,) + self.N)

    def sphere(self, F):
        F = F.reshape(F.shape[0], self.nr)
        x = torch.empty((F.shape[0], self.npw), dtype=torch.float64, device="cuda")
        f = F[:, self.ip]
        x[:, 0] = math.sqrt(self.omega) * F[:, 0].real
        x[:, 1::2] = math.sqrt(2 * self.omega) * f.real
        x[:, 2::2] = -math.sqrt(2 * self.omega) * f.imag
        return x

    def batched(self, f, x, n=64):
        return torch.cat([f(x[i:i + n]) for i in range(0, x.shape[0], n)])

    def to_grid(self, x):
        return self.batched(lambda y: (torch.fft.ifftn(self.coeffs(y), dim=(1, 2, 3)) * self.nr).real
                            .reshape(-1, self.nr), x)

    def from_grid(self, g):
        return self.batched(lambda y: self.sphere(torch.fft.fftn(y.reshape((-1,) + self.N),
                                                                 dim=(1, 2, 3)) / self.nr), g)

    def W(self, rho, pdep=True):
        def one(r):
            F = torch.fft.fftn(r.reshape((-1,) + self.N), dim=(1, 2, 3)) / self.nr
            x = (self.sphere(F) @ self.P) @ self.Pc.T if pdep else None
            F = F * self.vc
            if pdep:
                F += self.coeffs(x)
            return (torch.fft.ifftn(F, dim=(1, 2, 3)) * self.nr).real.reshape(-1, self.nr)

        return self.batched(one, rho)

    def proj(self, x):
        return x - (x @ self.phi.T) @ self.phi

    def pair_sum(self, L, M, xs):
        """out[b][v] = sum_u W(M_v L_u) xs[b][u] over all pairs of M = L."""
        out = torch.zeros_like(xs)
        for v in range(self.nv):
            w = self.W(L[v:] * M[v])
            for b in range(xs.shape[0]):
                out[b, v] += (w * xs[b, v:]).sum(0)
                out[b, v + 1:] += w[1:] * xs[b, v]
        return out

    def kernel_grid(self, ar):
        """s (v_c * Drho) phi_v - sum_v' tau_v'v a_v' for ar [b][v][r]."""
        z = -self.pair_sum(self.phir, self.phir, ar)
        for b in range(ar.shape[0]):
            z[b] += 2.0 * self.W((self.phir * ar[b]).sum(0)[None], False)[0] * self.phir
        return z

    def apply(self):
        A = torch.stack([self.proj(x) for x in self.X])
        ar = torch.stack([self.to_grid(a) for a in A])
        z = self.kernel_grid(ar)
        D = 0.5 * self.g2[None] - self.eps[:, None]
        for b in range(len(A)):
            z[b] += self.V.reshape(-1) * ar[b]
            A[b] = self.proj(self.from_grid(z[b]) + D * A[b])
        return A

    def u(self):
        A = self.proj(self.X)
        ar = self.to_grid(A)
        drho = (self.phir * ar).sum(0)
        g = 2.0 * self.W(drho[None], False)[0] * ar - self.pair_sum(ar, ar, self.phir[None])[0]
        S = self.phi @ self.from_grid(self.kernel_grid(ar[None])[0]).T
        return self.proj(self.from_grid(g)) - S @ A

    def coupling(self):
        out = []
        for x in self.X:
            ar = self.to_grid(self.proj(x))
            z = 2.0 * self.W((self.phir * ar).sum(0)[None], False)[0] * self.phir
            for v in range(self.nv):
                z[v] -= (self.W(ar * self.phir[v]) * self.phir).sum(0)
            out.append(self.proj(self.from_grid(z)))
        return torch.stack(out)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("zvector", "geometry"):
        return None  # iterative solves on the library's own ground state
    E = _Exact(case, seed)
    return E.apply() if kind == "apply" else E.u() if kind == "u" else E.coupling()
