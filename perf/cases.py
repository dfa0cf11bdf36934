"""The work users of this library have it do, as timed cases.

Each case is one call, or the few calls a program makes together, through the
public binding (paper_1207_2223_amd.wd): the operator alone, what a program
does with a new configuration, solves of one and of many right-hand sides on
the lattices of the benchmark and of the serving stream, solver sessions, the
molecular-dynamics force, trajectories and propagators.  Lattices range from
4^4 to 32^3 x 64, with extents that are no multiples of a work-group among
them.  Solves ask for a true residual of 1e-12, so that what is compared is the
solution and not the path the iteration took to it.
"""
import math
import os
import shutil
import tempfile

import torch

import paper_1207_2223_amd
from paper_1207_2223_amd import wd

DEVICE = "cuda"
PREC = {"f64": wd.WD_F64, "f32": wd.WD_F32, "f16": wd.WD_F16}
TOL = 1e-12
BETA = 5.6


def listed():
    return [
        # a small test lattice: the latency of one operator call
        dict(name="hop_4c4", kind="hop", Lx=4, Ly=4, Lz=4, Lt=4, prec="f64", recon=18, part="even", dagger=False, eps=0.3),
        # H on a whole lattice with ragged extents, FP16 storage inside
        dict(name="hop_full_ragged", kind="hop", Lx=10, Ly=14, Lz=6, Lt=22, prec="f16", recon=12, part="full", dagger=False, eps=0.5),
        # one parity block of the largest lattice, links with all 18 reals
        dict(name="hop_32c64", kind="hop", Lx=32, Ly=32, Lz=32, Lt=64, prec="f64", recon=18, part="odd", dagger=True, eps=0.5),
        # the normal operator of a user's own solver
        dict(name="normal_16c32", kind="normal", Lx=16, Ly=16, Lz=16, Lt=32, recon=12, eo=True, kappa=0.155, eps=0.5),
        # a new configuration: load it, its plaquette and Polyakov loop, one normal operator on the whole lattice
        dict(name="config_24c48", kind="config", Lx=24, Ly=24, Lz=24, Lt=48, recon=12, kappa=0.14, eps=0.5),
        # the smallest solve: FP64 CG on the full lattice
        dict(name="cg_full_4c4", kind="cg", Lx=4, Ly=4, Lz=4, Lt=4, prec="f64", recon=18, eo=False, nrhs=1, kappa=0.15, eps=0.3,
             tuned=False, delta=0.1),
        # eight right-hand sides together, default launch shapes
        dict(name="cg_16c32_8rhs", kind="cg", Lx=16, Ly=16, Lz=16, Lt=32, prec="f16", recon=12, eo=True, nrhs=8, kappa=0.155, eps=0.5,
             tuned=False, delta=0.1),
        # the benchmark's workload: twelve right-hand sides, tuned shapes
        dict(name="cg_32c64_12rhs", kind="cg", Lx=32, Ly=32, Lz=32, Lt=64, prec="f16", recon=12, eo=True, nrhs=12, kappa=0.156, eps=0.5,
             tuned=True, delta=0.01),
        # a serving step's life: requests join a session, are solved, and leave
        dict(name="session_12c24", kind="session", Lx=12, Ly=12, Lz=12, Lt=24, prec="f16", recon=18, nrhs=5, kappa=0.14, eps=0.5),
        # one molecular-dynamics force with its solve
        dict(name="force_16c32", kind="force", Lx=16, Ly=16, Lz=16, Lt=32, prec="f32", recon=12, kappa=0.14, eps=0.5),
        # a short trajectory that takes its proposal, as in thermalisation
        dict(name="hmc_8c16", kind="hmc", Lx=8, Ly=8, Lz=8, Lt=16, prec="f16", recon=12, kappa=0.14, eps=0.45, nsteps=5, chrono=1),
        # a point propagator and its pion correlator
        dict(name="propagator_16c16", kind="propagator", Lx=16, Ly=16, Lz=16, Lt=16, prec="f16", recon=12, kappa=0.14, eps=0.5),
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _extents(rng, vmax, vmin=256):
    """Even extents of 4 .. 64 with a volume near one drawn over its logarithm."""
    want = _log_uniform(rng, vmin, vmax)
    while True:
        L = [2 * round(_log_uniform(rng, 4, 48) / 2) for _ in range(3)]
        t = 2 * round(want / (L[0] * L[1] * L[2]) / 2)
        if 4 <= t <= 64 and vmin <= L[0] * L[1] * L[2] * t <= vmax:
            return dict(Lx=L[0], Ly=L[1], Lz=L[2], Lt=t)


def draw(rng):
    kind = rng.choice(["hop", "hop", "normal", "config", "cg", "cg", "session", "force", "hmc", "propagator"])
    eps = round(rng.uniform(0.3, 0.5), 3)
    c = dict(kind=kind, recon=rng.choice([12, 18]), eps=eps)
    # below the smallest critical hopping parameter of these fields, where the condition number is moderate on every draw
    kappa = round(rng.uniform(0.118, 0.126) if eps < 0.4 else rng.uniform(0.126, 0.134), 4)
    if kind == "hop":
        c.update(_extents(rng, 2 ** 21), prec=rng.choice(["f64", "f32", "f16"]), part=rng.choice(["even", "odd", "full"]),
                 dagger=rng.random() < 0.5)
    elif kind == "normal":
        c.update(_extents(rng, 2 ** 21), eo=rng.random() < 0.7, kappa=kappa)
    elif kind == "config":
        c.update(_extents(rng, 2 ** 20), kappa=kappa)
    elif kind == "cg":
        n = rng.randint(1, 12)
        eo = rng.random() < 0.8
        c.update(_extents(rng, 2 ** 21 // n), prec=rng.choice(["f64", "f32", "f16"]) if eo else "f64", eo=eo, nrhs=n, kappa=kappa,
                 tuned=False, delta=0.1)
    elif kind == "session":
        n = rng.randint(1, 8)
        c.update(_extents(rng, 2 ** 20 // n), prec=rng.choice(["f64", "f16"]), nrhs=n, kappa=kappa)
    elif kind == "force":
        c.update(_extents(rng, 2 ** 19), prec=rng.choice(["f64", "f32", "f16"]), kappa=kappa)
    elif kind == "hmc":
        c.update(_extents(rng, 2 ** 16), prec=rng.choice(["f64", "f16"]), kappa=kappa, nsteps=rng.randint(2, 6), chrono=rng.randint(0, 2))
    else:
        c.update(_extents(rng, 2 ** 17), prec=rng.choice(["f32", "f16"]), kappa=kappa)
    return c


def _dims(case):
    return tuple(case[k] for k in ("Lx", "Ly", "Lz", "Lt"))


# ---------------------------------------------------------------------------
# Inputs: U = exp(i eps H) per link, H = sum_a xi_a lambda_a / 2 with normal
# xi, re-unitarised; sources with Re, Im ~ N(0, 1/2); all from the seed alone.
# ---------------------------------------------------------------------------

def _links(V, eps, gen, device):
    """[V, 4, 3, 3] complex128 in SU(3)."""
    out = torch.empty((V, 4, 3, 3), dtype=torch.complex128, device=device)
    for mu in range(4):
        xi = torch.randn((8, V), dtype=torch.float64, device=device, generator=gen) * (0.5 * eps)
        r3 = 1 / math.sqrt(3.0)
        diag = [xi[2] + r3 * xi[7], -xi[2] + r3 * xi[7], -2 * r3 * xi[7]]
        up = {(0, 1): torch.complex(xi[0], -xi[1]), (0, 2): torch.complex(xi[3], -xi[4]), (1, 2): torch.complex(xi[5], -xi[6])}
        A = [[1j * (diag[i] if i == j else (up[i, j] if i < j else up[j, i].conj())) for j in range(3)] for i in range(3)]
        one = torch.ones(V, dtype=torch.complex128, device=device)
        E = [[one * (i == j) for j in range(3)] for i in range(3)]
        for n in range(20, 0, -1):  # exp(A) = 1 + A/1 (1 + A/2 (1 + ...)); two rows of it are enough
            E = [[(A[i][0] * E[0][j] + A[i][1] * E[1][j] + A[i][2] * E[2][j]) / n + (1.0 if i == j else 0.0) for j in range(3)] for i in range(3)]
        a, b = E[0], E[1]
        na = torch.sqrt(sum(z.abs() ** 2 for z in a))
        a = [z / na for z in a]
        ab = sum(x.conj() * y for x, y in zip(a, b))
        b = [y - ab * x for x, y in zip(a, b)]
        nb = torch.sqrt(sum(z.abs() ** 2 for z in b))
        b = [z / nb for z in b]
        c = [(a[(j + 1) % 3] * b[(j + 2) % 3] - a[(j + 2) % 3] * b[(j + 1) % 3]).conj() for j in range(3)]
        for i, row in enumerate((a, b, c)):
            for j in range(3):
                out[:, mu, i, j] = row[j]
    return out


def _sources(shape, gen, device):
    return torch.randn(shape, dtype=torch.complex128, device=device, generator=gen)


def _inputs(case, seed, device):
    dims = _dims(case)
    V = dims[0] * dims[1] * dims[2] * dims[3]
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed) * 7919 + 17)
    U = _links(V, case["eps"], gen, device)
    kind = case["kind"]
    if kind == "hop":
        n = V if case["part"] == "full" else V // 2
        return U, _sources((n, 4, 3), gen, device)
    if kind == "normal":
        return U, _sources((V // 2 if case["eo"] else V, 4, 3), gen, device)
    if kind == "config":
        return U, _sources((V, 4, 3), gen, device)
    if kind in ("cg", "session"):
        n = V // 2 if case.get("eo", True) else V
        return U, _sources((case["nrhs"], n, 4, 3), gen, device)
    if kind == "force":
        return U, _sources((V // 2, 4, 3), gen, device)
    return U, None


def _source_site(case):
    """A propagator's source: not the origin, on either parity."""
    return [(L // 2 + (1 if k == 0 else 0)) % L for k, L in enumerate(_dims(case))]


class State:
    """What a user's program holds before the call."""

    def __del__(self):
        sess = getattr(self, "sess", None)
        if sess is not None:
            wd.wd_session_destroy(sess)
            self.sess = None


_TABLE = None


def _shape_table():
    """The package's launch-shape table, as the benchmark uses it: a private copy, because the tuner appends to it."""
    global _TABLE
    if _TABLE is None:
        _TABLE = os.path.join(tempfile.mkdtemp(prefix="shapes_"), "table.txt")
        shutil.copy(os.path.join(os.path.dirname(paper_1207_2223_amd.__file__), "tune_mi355x.txt"), _TABLE)
        os.environ["WD_TUNE_CACHE"] = _TABLE


def prepare(case, seed):
    s = State()
    s.case = case
    kind = case["kind"]
    U, src = _inputs(case, seed, DEVICE)
    s.lat = wd.Lattice(_dims(case))
    s.src = src
    s.U = U
    if kind != "config":
        s.lat.gauge_load(U, recon=case["recon"])
    if kind in ("hop", "normal", "config", "cg"):
        s.out = torch.empty_like(src)
    if kind in ("cg", "session", "propagator"):
        s.params = wd.solver_params(tol=TOL, prec=PREC[case["prec"]], eo=1 if case.get("eo", True) else 0,
                                    delta=case.get("delta", 0.1), tuned=1 if case.get("tuned") else 0)
    if kind == "cg" and case["tuned"]:
        _shape_table()
        wd.wd_tune(s.lat.ctx, case["nrhs"], PREC[case["prec"]])
        wd.wd_tune(s.lat.ctx, case["nrhs"], wd.WD_F64)
    if kind == "session":
        s.sess = wd.wd_session_create(s.lat.ctx, case["nrhs"], s.params)
        s.out = torch.empty_like(src)
    if kind == "force":
        s.params = wd.solver_params(tol=TOL, prec=PREC[case["prec"]])
        s.out = torch.empty_like(U)
    if kind == "hmc":
        # the benchmark's molecular dynamics (force solves to 1e-8, the last one in FP64 to 1e-10), fewer steps
        force = wd.solver_params(tol=1e-8, prec=PREC[case["prec"]])
        last = wd.solver_params(tol=1e-10, prec=wd.WD_F64)
        s.hmc = wd.hmc_params(beta=BETA, kappa=case["kappa"], tau=0.02 * case["nsteps"], nsteps=case["nsteps"], seed=int(seed) + 1,
                              traj=3, force=force, h=last, metropolis=False, chrono=case["chrono"])
        s.now = torch.empty_like(U)
    if kind == "propagator":
        s.psi = torch.empty((12, s.lat.V, 4, 3), dtype=torch.complex128, device=DEVICE)
        s.at = _source_site(case)
    return s


def run(s):
    case, kind = s.case, s.case["kind"]
    if kind == "hop":
        part = {"full": wd.WD_FULL, "even": wd.WD_EVEN, "odd": wd.WD_ODD}[case["part"]]
        s.lat.dslash(s.out, s.src, part, dagger=1 if case["dagger"] else 0, prec=PREC[case["prec"]])
        return s.out
    if kind == "normal":
        s.lat.mdagm(s.out, s.src, case["kappa"], eo=1 if case["eo"] else 0)
        return s.out
    if kind == "config":
        s.lat.gauge_load(s.U, recon=case["recon"])
        plaq = s.lat.plaquette(s.U)
        loop = s.lat.polyakov(s.U)
        s.lat.mdagm(s.out, s.src, case["kappa"], eo=0)
        return {"plaquette": plaq, "loop_re": loop.real, "loop_im": loop.imag, "normal": s.out}
    if kind == "cg":
        status, _ = s.lat.cg_solve(s.out, s.src, case["kappa"], s.params)
        return {"x": s.out, "status": status}
    if kind == "session":
        slots = wd.wd_session_add(s.sess, s.src, case["kappa"])
        left = set(slots)
        while left:
            wd.wd_session_step(s.sess, 8)
            states, _ = wd.wd_session_poll(s.sess)
            for j in [j for j in left if states[j] == 2]:
                wd.wd_session_take(s.sess, j, s.out[slots.index(j)])
                left.discard(j)
        return s.out
    if kind == "force":
        wd.wd_md_force(s.lat.ctx, s.out, s.U, s.src, case["kappa"], BETA, s.params)
        return s.out
    if kind == "hmc":
        s.now.copy_(s.U)
        r = wd.hmc_trajectory(s.lat.ctx, s.now, s.hmc)
        return {"U": s.now, "plaquette": r["plaquette"], "H_old": r["H_old"], "H_new": r["H_new"], "accepted": r["accepted"]}
    status, _ = s.lat.point_propagator(s.psi, s.at, case["kappa"], s.params)
    return {"psi": s.psi, "corr": s.lat.pion_correlator(s.psi, s.at), "status": status}


# ---------------------------------------------------------------------------
# What a pass cannot do without
# ---------------------------------------------------------------------------

_SPINOR = {"f64": 192, "f32": 96, "f16": 52}
_HOP_FLOPS = 1320
# iterations of a solve to 1e-12 on these fields, about (the condition number sets them, not the code)
_ITERS = 150


def _solve_work(Vh, n, prec, eo, iters):
    """An iteration reads the links and streams each vector of its sweeps once."""
    sp, lk = _SPINOR[prec], 96 if prec == "f64" else 48
    sub = 1 if eo else 2
    per = 4 * 8 * lk + n * sp * (2 + 3 + 2 + 4 + 3)
    return iters * sub * Vh * per, iters * sub * Vh * n * 4 * _HOP_FLOPS


def work(case):
    dims, kind = _dims(case), case["kind"]
    V = dims[0] * dims[1] * dims[2] * dims[3]
    Vh = V // 2
    link = 16 * (9 if case["recon"] == 18 else 6)
    if kind == "hop":
        lk = link if case["prec"] == "f64" else 48
        n = V if case["part"] == "full" else Vh
        return dict(bytes=n * (8 * lk + 2 * 192), flops=n * _HOP_FLOPS)
    if kind == "normal":
        n = Vh if case["eo"] else V
        # two passes over the links for each of the two factors (even-odd: four half-volume sweeps), the vector in and out
        sweeps = 4 if case["eo"] else 2
        return dict(bytes=n * (sweeps * 8 * link + 2 * 192), flops=n * sweeps * _HOP_FLOPS)
    if kind == "config":
        # U once, each packed format written once; the operator as above; plaquette and loop on the U just read
        formats = link + 48 + 24 + 72 + 32
        return dict(bytes=V * (4 * (144 + formats) + 2 * 8 * link + 2 * 192), flops=V * (2 * _HOP_FLOPS + 6 * 3 * 198 + 198))
    if kind in ("cg", "session"):
        b, f = _solve_work(Vh, case["nrhs"], case["prec"], case.get("eo", True), _ITERS)
        return dict(bytes=b, flops=f)
    if kind == "force":
        b, f = _solve_work(Vh, 1, case["prec"], True, _ITERS)
        return dict(bytes=b + V * 4 * 144 * 2, flops=f + V * 4 * 3000)
    if kind == "hmc":
        b, f = _solve_work(Vh, 1, case["prec"], True, 90)
        b2, f2 = _solve_work(Vh, 1, "f64", True, 110)
        k = case["nsteps"] + 1
        return dict(bytes=k * (b + V * 4 * 144 * 3) + b2, flops=k * (f + V * 4 * 3000) + f2)
    b, f = _solve_work(Vh, 12, case["prec"], True, _ITERS)
    return dict(bytes=b + 12 * V * 192, flops=f + 12 * V * 2 * _HOP_FLOPS)


# ---------------------------------------------------------------------------
# The same in plain torch, complex128.  A spinor is [4][3] tensors over
# (right-hand side, t, z, y, x); the links [mu][a][b] tensors over (t, z, y, x).
# ---------------------------------------------------------------------------

# (1 + S gamma_mu) psi in the chiral basis: h0 = p0 + S f0 p[k0], h1 = p1 + S f1 p[k1]; row k0 = S g0 h0, row k1 = S g1 h1
_GAMMA = [((3, 1j), (2, 1j), (3, -1j), (2, -1j)),
          ((3, -1), (2, 1), (3, -1), (2, 1)),
          ((2, 1j), (3, -1j), (2, -1j), (3, 1j)),
          ((2, 1), (3, 1), (2, 1), (3, 1))]


def _grid(dims):
    return (dims[3], dims[2], dims[1], dims[0])


class _Plain:
    def __init__(self, dims, U):
        g = _grid(dims)
        self.g = g
        self.V = U.shape[0]
        self.u = [[[U[:, mu, a, b].reshape(g).contiguous() for b in range(3)] for a in range(3)] for mu in range(4)]
        ix = sum(torch.arange(n, device=U.device).view([-1 if q == k else 1 for q in range(4)]) for k, n in enumerate(g))
        self.par = (ix % 2).view(-1).bool()
        self.odd = (ix % 2).to(torch.float64)
        self.even = 1.0 - self.odd

    def field(self, v, parity=None):
        """[n, sites, 4, 3] to [4, 3, n, grid] (the other parity zero)."""
        n = v.shape[0]
        if parity is None:
            full = v
        else:
            full = torch.zeros((n, self.V, 4, 3), dtype=v.dtype, device=v.device)
            full[:, self.par == bool(parity)] = v
        return full.permute(2, 3, 0, 1).reshape((4, 3, n) + self.g).contiguous()

    def back(self, f, parity=None):
        n = f.shape[2]
        v = f.reshape(4, 3, n, self.V).permute(2, 3, 0, 1)
        return (v if parity is None else v[:, self.par == bool(parity)]).contiguous()

    def hop(self, psi, dagger=False):
        out = torch.zeros_like(psi)
        for mu in range(4):
            (k0, f0), (k1, f1), (_, g0), (_, g1) = _GAMMA[mu]
            dim = -1 - mu
            for fwd in (True, False):
                S = (-1 if fwd else 1) * (-1 if dagger else 1)
                h = torch.stack([psi[0] + S * f0 * psi[k0], psi[1] + S * f1 * psi[k1]])
                u = self.u[mu]
                if fwd:
                    h = torch.roll(h, -1, dims=dim)
                    w = torch.stack([sum(u[a][b] * h[:, b] for b in range(3)) for a in range(3)], dim=1)
                else:
                    w = torch.stack([sum(u[b][a].conj() * h[:, b] for b in range(3)) for a in range(3)], dim=1)
                    w = torch.roll(w, 1, dims=dim)
                out[0] += w[0]
                out[1] += w[1]
                out[k0] += (S * g0) * w[0]
                out[k1] += (S * g1) * w[1]
        return out

    def m(self, psi, kappa, dagger=False):
        return psi - kappa * self.hop(psi, dagger)

    def mhat(self, psi, kappa, dagger=False):
        """psi lives on the even sites: two hops bring it back there."""
        return psi - kappa * kappa * self.hop(self.hop(psi, dagger), dagger)

    def normal(self, psi, kappa, eo):
        f = self.mhat if eo else self.m
        return f(f(psi, kappa), kappa, True)

    def solve(self, b, kappa, eo, tol=1e-14):
        """CG on the normal operator, then one correction of the true residual."""
        dot = lambda a, c: (a.conj() * c).real.sum(dim=(0, 1, 3, 4, 5, 6), keepdim=True)  # noqa: E731
        x = torch.zeros_like(b)
        bb = dot(b, b)
        for goal in (1e-10, tol):
            r = b - self.normal(x, kappa, eo)
            p, rr = r.clone(), dot(r, r)
            for _ in range(3000):
                if bool((rr <= goal * goal * bb).all()):
                    break
                Ap = self.normal(p, kappa, eo)
                alpha = torch.where(rr > 0, rr / dot(p, Ap), torch.zeros_like(rr))
                x = x + alpha * p
                r = r - alpha * Ap
                new = dot(r, r)
                p = r + torch.where(rr > 0, new / rr, torch.zeros_like(rr)) * p
                rr = new
        return x


def _mat(a, b):
    return [[a[i][0] * b[0][j] + a[i][1] * b[1][j] + a[i][2] * b[2][j] for j in range(3)] for i in range(3)]


def _dag(a):
    return [[a[j][i].conj() for j in range(3)] for i in range(3)]


def _plaquettes(u):
    """sum over mu < nu of Re tr U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag / 3, per site."""
    at = lambda m, mu: [[torch.roll(z, -1, dims=-1 - mu) for z in row] for row in m]  # noqa: E731
    tot = 0
    for mu in range(4):
        for nu in range(mu + 1, 4):
            t = _mat(_mat(u[mu], at(u[nu], mu)), _dag(_mat(u[nu], at(u[mu], nu))))
            tot = tot + (t[0][0] + t[1][1] + t[2][2]).real / 3
    return tot


def _exact_force(dims, U, phi, kappa, beta):
    """dS/dt = sum tr(X F) for U -> exp(i t X) U, from the gradient of the action (at fixed solution X = A^-1 phi the fermion part
    changes as -|Mhat X|^2 does)."""
    X = _Plain(dims, U).solve(_Plain(dims, U).field(phi[None], 0), kappa, True)
    W = U.detach().clone().requires_grad_(True)
    p = _Plain(dims, W)
    with torch.enable_grad():
        S = beta * (6.0 * p.V - _plaquettes(p.u).sum()) - p.mhat(X, kappa).abs().square().sum()
        (G,) = torch.autograd.grad(S, W)
    F = 1j * (U[..., :, :, None] * G.conj().transpose(-1, -2)[..., None, :, :]).sum(-2)
    F = 0.5 * (F + F.conj().transpose(-1, -2))
    tr = (F[..., 0, 0] + F[..., 1, 1] + F[..., 2, 2]) / 3
    return F - tr[..., None, None] * torch.eye(3, dtype=F.dtype, device=F.device)


def exact(case, seed, device=None):
    dims, kind = _dims(case), case["kind"]
    V = dims[0] * dims[1] * dims[2] * dims[3]
    n = case.get("nrhs", 12 if kind == "propagator" else 1)
    if kind == "hmc" or (kind in ("cg", "session", "propagator", "force") and V * n > 2 ** 20 + 2 ** 19):
        return None
    U, src = _inputs(case, seed, device or DEVICE)
    if kind == "force":
        return _exact_force(dims, U, src, case["kappa"], BETA)
    p = _Plain(dims, U)
    if kind == "hop":
        if case["part"] == "full":
            return p.back(p.hop(p.field(src[None]), case["dagger"]))[0]
        odd = case["part"] == "odd"
        return p.back(p.hop(p.field(src[None], not odd), case["dagger"]), odd)[0]
    if kind == "normal":
        par = 0 if case["eo"] else None
        return p.back(p.normal(p.field(src[None], par), case["kappa"], case["eo"]), par)[0]
    if kind == "config":
        loop = p.u[3]
        line = [[loop[i][j][0] for j in range(3)] for i in range(3)]
        for t in range(1, dims[3]):
            line = _mat(line, [[loop[i][j][t] for j in range(3)] for i in range(3)])
        tr = complex(((line[0][0] + line[1][1] + line[2][2]) / 3).mean())
        return {"plaquette": float(_plaquettes(p.u).sum()) / (6.0 * V), "loop_re": tr.real, "loop_im": tr.imag,
                "normal": p.back(p.normal(p.field(src[None]), case["kappa"], False))[0]}
    if kind in ("cg", "session"):
        par = 0 if case.get("eo", True) else None
        x = p.back(p.solve(p.field(src, par), case["kappa"], par is not None), par)
        return {"x": x, "status": None} if kind == "cg" else x
    # M psi = b as Mhat psi_e = b_e + kappa D_eo b_o, psi_o = b_o + kappa D_oe psi_e
    at = _source_site(case)
    lex = at[0] + dims[0] * (at[1] + dims[1] * (at[2] + dims[2] * at[3]))
    b = torch.zeros((12, V, 4, 3), dtype=torch.complex128, device=U.device)
    for j in range(12):
        b[j, lex, j // 3, j % 3] = 1
    b = p.field(b)
    bo, k = b * p.odd, case["kappa"]
    be = b * p.even + k * p.hop(bo)
    xe = p.solve(p.mhat(be, k, True), k, True)
    psi = xe + bo + k * p.hop(xe) * p.odd
    slices = psi.abs().square().sum(dim=(0, 1, 2, 4, 5, 6))
    return {"psi": p.back(psi), "corr": torch.roll(slices, -at[3]), "status": None}
