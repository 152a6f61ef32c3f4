"""Timed workloads of the library, through its public Python entry points.

Every case is one call (or the short sequence of calls) that a ChFSI program
makes again and again: the operator on a block, the Chebyshev filter in its
forms and precisions, the orthonormalisation, the Rayleigh-Ritz step with the
densities, the spectral bound, the adjoint of the filter, a batch of small
systems, new local fields, and whole SCF iterations.  Meshes follow the
synthetic systems of this repository: cells of 1.2 bohr, Gaussian wells of the
same number per volume, a field B_xc of 0.1 Ha, pseudo-atoms with s, p (and d)
projectors.

`prepare` builds what a program holds before the call (operator handle, fields,
blocks), `run` is one pass, `work` the bytes and operations that it cannot do
without, `exact` the same outputs from plain torch in 64 bits.
"""
import math

import numpy as np
import torch

import paper_2410_02754_amd as chfsi
from paper_2410_02754_amd import autograd as chfsi_autograd

H_CELL = 1.2                      # bohr, cell edge of every mesh
KT = 500 * 3.166811563e-6         # Ha, the smearing of the densities
A_CUT, A_LOW = 8.0, -6.0          # Ha: the filter damps [A_CUT, b] and scales at A_LOW


def _case(kind, cells, p, vec, **kw):
    nx, ny, nz = (cells,) * 3 if isinstance(cells, int) else cells
    n = nx * ny * nz
    c = {"kind": kind, "nx": nx, "ny": ny, "nz": nz, "p": p, "vec": vec, "lmax": 1, "atoms": max(1, n // 64), "k": 0.0,
         "form": "cell", "prec": "fp64", "degree": 1}
    c.update(kw)
    return c


def listed():
    return [
        # one product with H on a small block of a small system: launches and latency
        _case("apply", 3, 4, 32, name="apply_small", atoms=2),
        # the filter of one 128-column block with stored cell matrices at Gamma, p = 6, d projectors
        _case("filter", 8, 6, 128, name="filter_cell_fp64", lmax=2, atoms=4, degree=24),
        # the filter with single-precision products at a k-point, ragged block width
        _case("filter", 10, 5, 200, name="filter_cell_mixed_k", prec="mixed", k=0.21, degree=16, atoms=16),
        # the filter with the matrix-free operator on a large mesh at Gamma
        _case("filter", 16, 6, 128, name="filter_mf_fp64", form="matrix_free", lmax=2, atoms=33, degree=24),
        # the residual form with single-precision products, odd cell counts, a k-point
        _case("resid", 9, 5, 130, name="filter_resid_mf_mixed_k", form="matrix_free", prec="mixed", k=0.18, degree=16,
              atoms=12),
        # orthonormalisation of the whole block of a k-point
        _case("chol", 12, 5, 384, name="chol_gs_384", atoms=0),
        # Rayleigh-Ritz of the whole block, occupations and densities
        _case("ritz", 10, 5, 256, name="ritz_density_256", form="matrix_free", k=0.15, atoms=16),
        # spectral bounds before a filter: many single-column products, each waited for
        _case("lanczos", 10, 5, 1, name="lanczos_bounds", form="matrix_free", degree=20, atoms=16),
        # gradients through the filter with respect to the block and the fields
        _case("adjoint", 8, 5, 128, name="filter_adjoint", form="matrix_free", degree=16, atoms=4),
        # many small systems filtered together
        _case("batch", 3, 4, 32, name="batch_small", atoms=2, degree=10, tasks=32),
        # new fields in an operator with stored cell matrices at two k-points, and a first product with it
        _case("fields", 8, 5, 16, name="new_fields", k=0.2, atoms=8),
        # SCF iterations of a small system: every step of the loop
        _case("scf", 4, 4, 32, name="scf_small", atoms=2, degree=10),
    ]


def draw(rng):
    """One more case of the same ranges; sizes over their logarithm, odd ones among them."""
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["apply", "filter", "filter", "filter", "resid", "chol", "ritz", "lanczos", "adjoint", "batch",
                       "fields", "scf"])
    p = rng.choice([3, 4, 5, 5, 6, 6, 7])
    form = rng.choice(["cell", "matrix_free"])
    prec = rng.choice(["fp64", "mixed"])
    k = rng.choice([0.0, round(rng.uniform(0.05, 0.3), 4)])
    lmax = rng.choice([0, 1, 1, 2])
    degree = rng.randint(4, 24)
    # nodes of the mesh per direction, so that a high degree goes with fewer cells
    if kind in ("batch", "scf"):
        p, top, vec = min(p, 5), 18, log_int(12, 48)
    elif kind == "apply":
        top, vec = 40, log_int(1, 64)
    elif kind == "fields":
        top, vec = 40, log_int(4, 24)
    elif kind in ("chol", "ritz"):
        top, vec = 50, log_int(24, 400)
    else:
        top, vec = (64 if form == "matrix_free" and kind != "adjoint" else 44), log_int(20, 200)
    cells = tuple(max(2, log_int(max(2, top / p / 4), top / p)) for _ in range(3))
    vec = max(1, min(vec, cells[0] * cells[1] * cells[2] * p ** 3 // 4))       # far fewer columns than unknowns
    c = _case(kind, cells, p, vec, form=form, prec=prec, k=k, lmax=lmax, degree=degree)
    if kind in ("ritz", "chol", "lanczos", "adjoint", "scf", "fields"):
        c["prec"] = "fp64"
    if kind == "fields":
        c["form"] = "cell"
    if kind == "chol":
        c.update(atoms=0, k=0.0, form="cell")
    if kind == "lanczos":
        c.update(vec=1, degree=rng.randint(8, 20))
    if kind == "batch":
        c.update(tasks=log_int(4, 24), form="cell", degree=rng.randint(4, 12))
    if kind == "scf":
        c.update(degree=rng.randint(6, 12), k=0.0)
    return c


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------
class Atom:
    """The fields of the library's atom description."""

    def __init__(self, pos, lmax):
        self.pos, self.lmax = tuple(float(x) for x in pos), int(lmax)
        self.sigma, self.rcut = 0.7, 4.2
        self.d0, self.dso = (1.0, 0.5, 0.25)[:self.lmax + 1], 0.05


class System:
    """Mesh, fields and atoms of a case, from the seed alone."""

    def __init__(self, case, seed):
        rng = np.random.default_rng([int(seed), 77])
        self.nc = (case["nx"], case["ny"], case["nz"])
        self.box = tuple(H_CELL * n for n in self.nc)
        self.p, self.np1 = case["p"], case["p"] + 1
        k = case["k"]
        self.kpts = [(k, -0.7 * k, 0.4 * k)] if case["kind"] != "fields" else [(0.0, 0.0, 0.0), (k, -0.7 * k, 0.4 * k)]
        self.k = np.array(self.kpts[-1])
        vol = float(np.prod(self.box))
        G = max(2, round(200 / 24.0 ** 3 * vol))
        self.centres = rng.uniform(size=(G, 3)) * self.box
        self.amps = rng.uniform(-2.0, 0.0, size=G)
        self.bcen = rng.uniform(size=(3, 3)) * self.box
        d = rng.normal(size=(3, 3))
        self.bdir = d / np.linalg.norm(d, axis=1, keepdims=True)
        self.atoms = [Atom(rng.uniform(size=3) * self.box, case["lmax"]) for _ in range(case["atoms"])]
        self.E = int(np.prod(self.nc))
        self.Nd = tuple(n * self.p for n in self.nc)
        self.n_dof = 2 * int(np.prod(self.Nd))
        self.xq, self.wq = np.polynomial.legendre.leggauss(self.np1)

    def axis_points(self, d):
        """Quadrature points along direction d, cell by cell."""
        return ((np.arange(self.nc[d])[:, None] + 0.5 * (self.xq + 1.0)[None, :]) * H_CELL).reshape(-1)

    def _separable(self, centres, weights, width):
        """sum_g w_g exp(-|r - c_g|^2 / 2 width^2) over periodic images, on the tensor grid [z][y][x]."""
        f = []
        for d in range(3):
            x, L = self.axis_points(d), self.box[d]
            n = int(math.ceil(9.0 * width / L)) + 1
            t = sum(np.exp(-(x[None, :] - centres[:, d:d + 1] - i * L) ** 2 / (2 * width ** 2)) for i in range(-n, n + 1))
            f.append(torch.tensor(t, device="cuda"))
        w = torch.tensor(weights, device="cuda")
        out = [torch.matmul((w[:, j, None, None] * f[2][:, :, None] * f[1][:, None, :]).reshape(len(w), -1).T, f[0])
               for j in range(w.shape[1])]
        return torch.stack(out, -1).reshape(f[2].shape[1], f[1].shape[1], f[0].shape[1], -1)

    def cellwise(self, t):
        """[z][y][x][c] on the tensor grid -> [cell][point][c] in the library's order."""
        n = self.np1
        nx, ny, nz = self.nc
        return t.reshape(nz, n, ny, n, nx, n, -1).permute(0, 2, 4, 1, 3, 5, 6).reshape(self.E, n ** 3, -1).contiguous()

    def fields(self):
        V = self.cellwise(self._separable(self.centres, self.amps[:, None], 1.0))[..., 0].contiguous()
        v = self._separable(self.bcen, self.bdir, 2.0)
        v[..., 2] += 0.5
        return V, self.cellwise(0.1 * v / v.norm(dim=-1, keepdim=True))

    def bound(self):
        """An upper bound of the spectrum of the scaled operator from its 1-D kinetic parts."""
        r = Reference1D(self.p)
        top = sum(0.5 * (math.sqrt(2.0 * r.kinetic_top(n)) + abs(k)) ** 2 for n, k in zip(self.nc, self.k))
        return 1.02 * top + 12.0

    def random_block(self, seed, n):
        g = torch.Generator(device="cuda").manual_seed(int(seed))
        x = torch.rand((self.n_dof, n, 2), generator=g, device="cuda", dtype=torch.float64)
        return torch.view_as_complex(x.mul_(2.0).sub_(1.0))

    def smooth_block(self, seed, n):
        """Columns like those after a few passes: the lowest plane waves with random spins, and a little noise."""
        rng = np.random.default_rng([int(seed), 5])
        m = 1
        while (2 * m + 1) ** 3 < n:
            m += 1
        G = np.array([(i, j, l) for l in range(-m, m + 1) for j in range(-m, m + 1) for i in range(-m, m + 1)])
        kin = 0.5 * ((2 * np.pi * G / np.array(self.box) + self.k) ** 2).sum(1)
        G = G[np.argsort(kin, kind="stable")[:n]]
        gll = Reference1D(self.p).xi
        ph = []
        for d in range(3):
            x = ((np.arange(self.nc[d])[:, None] + 0.5 * (gll[:-1] + 1.0)[None, :]) * H_CELL).reshape(-1)
            e = np.exp(2j * np.pi * x[:, None] * G[None, :, d] / self.box[d])
            ph.append(torch.tensor(e, device="cuda"))
        X = 0.02 * self.random_block(seed, n)
        spin = rng.normal(size=(2, n)) + 1j * rng.normal(size=(2, n))
        spin = torch.tensor(spin / np.linalg.norm(spin, axis=0), device="cuda")
        W = ph[2][:, None, None] * ph[1][None, :, None] * ph[0][None, None]
        return X.reshape(-1, 2, n).add_(W.reshape(-1, 1, n) * spin[None]).reshape(-1, n), np.sort(kin)[:n]


def orthonormal(X):
    """X with orthonormal columns, in plain torch."""
    S = (X.mH @ X).cpu()
    L = torch.linalg.cholesky(S)
    R = torch.linalg.solve_triangular(L, torch.eye(len(S), dtype=S.dtype), upper=False).mH
    return X @ R.to(X.device)


def _operator(s, case, stream=None, fields=None):
    op = chfsi.Operator(s.nc, s.box, s.p, "gl", s.np1, s.kpts, stream=stream, form=case["form"])
    V, B = s.fields() if fields is None else fields
    op.set_local(V, B)
    if s.atoms:
        op.set_atoms(s.atoms)
    return op, V, B


def prepare(case, seed):
    kind, n = case["kind"], case["vec"]
    s = System(case, seed)
    st = {"case": case, "bounds": (A_CUT, s.bound(), A_LOW), "ik": 0}
    if kind == "batch":
        stream = torch.cuda.Stream()
        st["stream"] = stream
        with torch.cuda.stream(stream):
            st["ops"], systems = [], [System(case, 1000 * seed + t) for t in range(case["tasks"])]
            rows = s.n_dof
            st["X0"] = torch.cat([y.random_block(1000 * seed + t, n) for t, y in enumerate(systems)])
            st["X"], st["W"] = st["X0"].clone(), torch.empty_like(st["X0"])
            tasks = []
            for t, y in enumerate(systems):
                op = _operator(y, case, stream.cuda_stream)[0]
                st["ops"].append(op)
                tasks.append((op, 0, st["X"][t * rows:(t + 1) * rows], st["W"][t * rows:(t + 1) * rows]))
            st["batch"] = chfsi.Batch(tasks, case["degree"], prec=case["prec"])
            stream.synchronize()
        return st
    if kind == "scf":
        op = chfsi.Operator(s.nc, s.box, s.p, "gl", s.np1, s.kpts, form=case["form"])
        op.set_atoms(s.atoms)
        V, B = s.fields()
        rho = torch.rand(V.shape, generator=torch.Generator(device="cuda").manual_seed(seed), device="cuda",
                         dtype=torch.float64)
        st["ne"] = 0.8 * n
        st["rho0"] = (1.0 + 0.3 * rho) * (st["ne"] / float(np.prod(s.box)) / 1.15)
        st["m0"] = 0.1 * st["rho0"][..., None] * (B / B.norm(dim=-1, keepdim=True))
        st.update(op=op, V=V, B=B, seed=seed, X=torch.empty((s.n_dof, n), dtype=torch.complex128, device="cuda"))
        for k in ("rho", "rho_out"):
            st[k] = torch.empty_like(st["rho0"])
        for k in ("m", "m_out"):
            st[k] = torch.empty_like(st["m0"])
        return st
    if kind == "chol":
        st["op"] = chfsi.Operator(s.nc, s.box, s.p, "gl", s.np1, s.kpts)
        st["X"] = s.random_block(seed, n)
        return st
    op, V, B = _operator(s, case)
    st["op"] = op
    if kind in ("ritz", "resid"):
        st["X"], theta = s.smooth_block(seed, n)
    elif kind != "lanczos":
        st["X"] = s.random_block(seed, n)
    if kind in ("apply", "filter", "ritz", "fields"):
        st["W"] = torch.empty_like(st["X"])
    if kind == "filter":
        st["Y"] = torch.empty_like(st["X"])
    elif kind == "resid":
        # Ritz values and residuals of a block that is nearly converged
        st["theta"] = np.ascontiguousarray(theta)
        st["R"] = s.random_block(seed + 1, n).mul_(0.02)
        st["Y"] = torch.empty_like(st["X"])
        st["W"] = torch.empty((s.n_dof, 2 * n), dtype=torch.complex128, device="cuda")
    elif kind == "ritz":
        st["X"] = orthonormal(st["X"])
        st["rho"] = torch.zeros_like(V)
        st["mag"] = torch.zeros_like(B)
    elif kind == "lanczos":
        st["v0"] = s.random_block(seed, 1)[:, 0].contiguous()
    elif kind == "adjoint":
        st["X"].requires_grad_(True)
        st["V"], st["B"] = V.requires_grad_(True), B.requires_grad_(True)
        st["G"] = s.random_block(seed + 2, n)
    elif kind == "fields":
        st["V"], st["B"], st["ik"] = V, B, 1
    return st


# --------------------------------------------------------------------------
# One pass
# --------------------------------------------------------------------------
def run(st):
    case = st["case"]
    kind, m = case["kind"], case["degree"]
    a, b, a0 = st["bounds"]
    if kind == "apply":
        return st["op"].apply_H(st["X"], st["W"], prec=case["prec"]).to(_carried(case))
    if kind == "filter":
        # the program keeps its Ritz block and filters a copy
        st["Y"].copy_(st["X"])
        st["op"].cheb_filter(st["Y"], st["W"], m, a, b, a0, prec=case["prec"])
        return st["Y"].to(_carried(case))
    if kind == "resid":
        st["Y"].copy_(st["X"])
        st["op"].cheb_filter_resid(st["Y"], st["R"], st["theta"], st["W"], m, a, b, a0, prec=case["prec"])
        return st["Y"].to(_carried(case))
    if kind == "chol":
        return st["op"].chol_gs(st["X"])
    if kind == "ritz":
        # the rotated block is left out: its columns' phases are the eigensolver's choice; the densities are
        # those of the rotated block
        theta, resid = st["op"].rayleigh_ritz(st["X"], st["W"])
        occ, _, _ = chfsi.fermi_dirac(theta, 0.8 * case["vec"], KT)
        st["rho"].zero_()
        st["mag"].zero_()
        st["op"].density(st["X"], occ, st["rho"], st["mag"])
        return theta, resid, occ, st["rho"], st["mag"]
    if kind == "lanczos":
        return st["op"].lanczos_bounds(st["v0"], m)
    if kind == "adjoint":
        Y = chfsi_autograd.cheb_filter(st["X"], st["V"], st["B"], st["op"], m, a, b, a0)
        return (Y.detach(),) + torch.autograd.grad(Y, (st["X"], st["V"], st["B"]), st["G"])
    if kind == "batch":
        with torch.cuda.stream(st["stream"]):
            st["X"].copy_(st["X0"])
            st["batch"].filter(a, b, a0)
        if case["prec"] == "fp64":
            return st["X"]
        with torch.cuda.stream(st["stream"]):
            return st["X"].to(torch.complex64)
    if kind == "fields":
        st["op"].set_local(st["V"], st["B"])
        return st["op"].apply_H(st["X"], st["W"], ik=st["ik"])
    if kind == "scf":
        st["rho"].copy_(st["rho0"])
        st["m"].copy_(st["m0"])
        hist, theta, occ, _ = chfsi.scf_run(
            st["op"], st["V"], st["B"], st["rho"], st["m"], st["rho_out"], st["m_out"], st["X"], st["ne"], 10 * KT, m,
            passes_first=2, max_iter=3, alpha=0.4, k0=0.8, tol=1e-12, seed=st["seed"], bounds=[b] * 3)
        return {"rho": st["rho"], "m": st["m"], "rho_out": st["rho_out"], "m_out": st["m_out"], "theta": theta, "occ": occ,
                "resid": [h["resid"] for h in hist], "mu": [h["mu"] for h in hist]}
    raise KeyError(kind)


def _carried(case):
    """The type in which a block goes on: products in single precision leave that many digits."""
    return torch.complex128 if case["prec"] == "fp64" else torch.complex64


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    kind, n, p, m = case["kind"], case["vec"], case["p"], case["degree"]
    E = case["nx"] * case["ny"] * case["nz"]
    dof, np1 = 2 * E * p ** 3, p + 1
    block = 16.0 * dof * n
    size = 8 if case["prec"] == "fp64" else 4
    gamma = case["k"] == 0.0
    # one product with H: the cell operators (or 32 bytes a quadrature point) once, the block in and out
    if case["form"] == "cell" and kind != "lanczos":
        op_b = E * (4.0 if gamma else 5.0) * np1 ** 6 * size
        op_f = E * (8 if gamma else 12) * 2.0 * np1 ** 6 * n
    else:
        op_b = E * 4.0 * np1 ** 3 * size
        op_f = E * 2 * 9 * 2 * 2.0 * (np1 ** 4 / 2.0) * n
    sup = min(1.0, 4.0 / 3.0 * math.pi * 4.2 ** 3 / (E * H_CELL ** 3)) * dof * case["atoms"]
    pj = (case["lmax"] + 1) ** 2
    op_f += 2 * (4 if gamma else 8) * sup * pj * n
    op_b += sup / 2 * pj * 16
    apply_b, apply_f = op_b + 2 * block, op_f
    step_b = op_b + 3 * block            # a recurrence step reads two blocks and writes one
    if kind == "apply":
        b, f = apply_b, apply_f
    elif kind == "filter":
        b, f = m * step_b, m * apply_f
    elif kind == "resid":
        b, f = (m - 1) * (step_b + block), (m - 1) * apply_f
    elif kind == "chol":
        b, f = 3 * block, 8.0 * dof * n * n
    elif kind == "ritz":
        b, f = apply_b + 6 * block, apply_f + (4 + 16) * dof * float(n) * n
    elif kind == "lanczos":
        b, f = m * (op_b + 3 * block), m * apply_f
    elif kind == "adjoint":
        b, f = 3 * m * step_b, 3 * m * apply_f
    elif kind == "batch":
        b, f = case["tasks"] * m * step_b, case["tasks"] * m * apply_f
    elif kind == "fields":
        b, f = 2 * op_b * 1.5 + apply_b, apply_f + E * 4 * 2 * 2.0 * np1 ** 7
    else:
        b, f = (5 * m + 12) * step_b, (5 * m + 8) * apply_f
    return {"bytes": float(b), "flops": float(f)}


# --------------------------------------------------------------------------
# The same outputs from plain torch
# --------------------------------------------------------------------------
class Reference1D:
    """Gauss-Lobatto-Legendre nodes of degree p and the Lagrange basis at the Gauss points."""

    def __init__(self, p):
        c = np.zeros(p + 1)
        c[p] = 1.0
        P = np.polynomial.legendre.Legendre(c)
        x = np.sort(np.concatenate([[-1.0], np.real(P.deriv().roots()), [1.0]]))
        for _ in range(3):                       # Newton steps on P'(x) = 0 for the inner nodes
            x[1:-1] -= P.deriv()(x[1:-1]) / P.deriv(2)(x[1:-1])
        x = 0.5 * (x - x[::-1])
        self.xi, self.w = x, 2.0 / (p * (p + 1) * P(x) ** 2)
        self.xq, self.wq = np.polynomial.legendre.leggauss(p + 1)
        self.B, self.D = self.basis(self.xq)

    def basis(self, y):
        """l_a(y), l_a'(y) as [a][point]."""
        x, n = self.xi, len(self.xi)
        B, D = np.ones((n, len(y))), np.zeros((n, len(y)))
        for a in range(n):
            for j in range(n):
                if j != a:
                    B[a] *= (y - x[j]) / (x[a] - x[j])
            for i in range(n):
                if i != a:
                    t = np.full(len(y), 1.0 / (x[a] - x[i]))
                    for j in range(n):
                        if j != a and j != i:
                            t *= (y - x[j]) / (x[a] - x[j])
                    D[a] += t
        return B, D

    def kinetic_top(self, cells):
        """Largest eigenvalue of -u''/2 on `cells` periodic cells with the lumped mass."""
        p, N = len(self.xi) - 1, cells * (len(self.xi) - 1)
        K, M = np.zeros((N, N)), np.zeros(N)
        Ke = 0.5 * (2.0 / H_CELL) * (self.D * self.wq) @ self.D.T
        for c in range(cells):
            g = (c * p + np.arange(p + 1)) % N
            np.add.at(K, (g[:, None], g[None, :]), Ke)
            np.add.at(M, g, self.w * H_CELL / 2)
        s = 1.0 / np.sqrt(M)
        return float(np.linalg.eigvalsh(K * s[:, None] * s[None, :])[-1])


def _harmonics(lmax, d):
    """r^l Y_lm as a list, in the library's order."""
    x, y, z = d[..., 0], d[..., 1], d[..., 2]
    out = [np.full(x.shape, 0.5 / math.sqrt(math.pi))]
    if lmax >= 1:
        c = math.sqrt(3.0 / (4.0 * math.pi))
        out += [c * x, c * y, c * z]
    if lmax >= 2:
        c = 0.5 * math.sqrt(15.0 / math.pi)
        out += [c * x * y, c * y * z, 0.25 * math.sqrt(5.0 / math.pi) * (2 * z * z - x * x - y * y), c * x * z,
                0.5 * c * (x * x - y * y)]
    return out


def _delta(atom):
    """D0 within each shell and dso L.S, index 2 chi + spin."""
    sig = np.array([[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]], dtype=complex)
    eps = np.zeros((3, 3, 3))
    for i, j, l in ((0, 1, 2), (1, 2, 0), (2, 0, 1)):
        eps[i, j, l], eps[i, l, j] = 1.0, -1.0
    L1 = -1j * eps                               # (L_c)_{ba} on (x, y, z)
    r2, r6 = 1 / math.sqrt(2.0), 1 / math.sqrt(6.0)
    T = np.zeros((5, 3, 3))                      # the d harmonics as traceless symmetric tensors
    T[0, 0, 1] = T[0, 1, 0] = T[1, 1, 2] = T[1, 2, 1] = T[3, 0, 2] = T[3, 2, 0] = r2
    T[2] = np.diag([-r6, -r6, 2 * r6])
    T[4] = np.diag([r2, -r2, 0.0])
    L2 = np.array([[[np.sum(T[m] * (L1[c] @ T[q] + T[q] @ L1[c].T)) for q in range(5)] for m in range(5)]
                   for c in range(3)])
    n = (atom.lmax + 1) ** 2
    out, o = np.zeros((2 * n, 2 * n), dtype=complex), 0
    for l in range(atom.lmax + 1):
        w = 2 * (2 * l + 1)
        D = atom.d0[l] * np.eye(w, dtype=complex)
        for c in range(3 if l else 0):
            D += atom.dso * 0.5 * np.kron((L1, L2)[l - 1][c], sig[c])
        out[o:o + w, o:o + w] = D
        o += w
    return out


class Reference:
    """The scaled Hamiltonian as plain tensor operations in 64 bits."""

    def __init__(self, s, V, B):
        dev = "cuda"
        r = Reference1D(s.p)
        n, nc, p = s.np1, s.nc, s.p
        self.s, self.n = s, n
        idx = [((np.arange(nc[d])[:, None] * p + np.arange(n)[None, :]) % s.Nd[d]) for d in range(3)]
        g = (idx[0][None, None, :, None, None, :] + s.Nd[0] * (idx[1][None, :, None, None, :, None]
             + s.Nd[1] * idx[2][:, None, None, :, None, None]))
        self.nodes = torch.tensor(np.broadcast_to(g, (nc[2], nc[1], nc[0], n, n, n)).reshape(s.E, n ** 3).copy(),
                                  device=dev)
        self.M = s.n_dof // 2
        w = r.w * H_CELL / 2
        w3 = torch.tensor((w[:, None, None] * w[None, :, None] * w[None, None, :]).reshape(-1), device=dev)
        mass = torch.zeros(self.M, dtype=torch.float64, device=dev)
        mass.index_add_(0, self.nodes.reshape(-1), w3.repeat(s.E))
        self.sc = mass.rsqrt()
        q = r.wq * H_CELL / 2
        self.wJ = torch.tensor((q[:, None, None] * q[None, :, None] * q[None, None, :]).reshape(-1), device=dev)
        self.B = torch.tensor(r.B, device=dev)
        self.D = torch.tensor(r.D * 2.0 / H_CELL, device=dev)
        self.V, self.Bf = V, B
        self.k = [float(x) for x in s.k]
        self.proj = [self._projector(a, r) for a in s.atoms]

    def _projector(self, atom, r):
        """(support nodes, scaled projector values on them, coupling) of one atom."""
        s, n = self.s, self.n
        ax = [s.axis_points(d).reshape(s.nc[d], n) for d in range(3)]
        cand = []
        for d in range(3):
            near = np.zeros(s.nc[d], dtype=bool)
            img = int(math.ceil(atom.rcut / s.box[d])) + 1
            for i in range(-img, img + 1):
                c = atom.pos[d] + i * s.box[d]
                lo = np.arange(s.nc[d]) * H_CELL
                near |= (lo < c + atom.rcut) & (lo + H_CELL > c - atom.rcut)
            cand.append(np.nonzero(near)[0])
        cz, cy, cx = (t.reshape(-1) for t in np.meshgrid(cand[2], cand[1], cand[0], indexing="ij"))
        cells = cx + s.nc[0] * (cy + s.nc[1] * cz)
        C = len(cells)
        pts = np.empty((C, n, n, n, 3))
        pts[..., 0] = ax[0][cx][:, None, None, :]
        pts[..., 1] = ax[1][cy][:, None, :, None]
        pts[..., 2] = ax[2][cz][:, :, None, None]
        beta = np.zeros((C, n, n, n, (atom.lmax + 1) ** 2), dtype=complex)
        img = [int(math.ceil(atom.rcut / L)) for L in s.box]
        for iz in range(-img[2], img[2] + 1):
            for iy in range(-img[1], img[1] + 1):
                for ix in range(-img[0], img[0] + 1):
                    sh = np.array([ix, iy, iz]) * s.box
                    d = pts - np.array(atom.pos) - sh
                    r2 = (d * d).sum(-1)
                    hit = r2 < atom.rcut ** 2
                    if not hit.any():
                        continue
                    dd, g = d[hit], np.exp(-r2[hit] / (2 * atom.sigma ** 2))
                    ph = np.exp(-1j * ((pts[hit] - sh) @ s.k))
                    col, h = 0, _harmonics(atom.lmax, dd)
                    vals = np.empty((len(dd), len(h)), dtype=complex)
                    for l in range(atom.lmax + 1):
                        cl = math.sqrt(2.0 / (math.gamma(l + 1.5) * atom.sigma ** (2 * l + 3)))
                        for _ in range(2 * l + 1):
                            vals[:, col] = ph * cl * g * h[col]
                            col += 1
                    beta[hit] += vals
        F = torch.tensor(beta, device="cuda").reshape(C, n ** 3, -1) * self.wJ[None, :, None]
        F = torch.view_as_real(F).reshape(C, n, n, n, -1)
        F = torch.einsum("czyxf,az,by,dx->cabdf", F, self.B, self.B, self.B)
        F = torch.view_as_complex(F.reshape(C * n ** 3, -1, 2).contiguous())
        where = self.nodes[torch.tensor(cells, device="cuda")].reshape(-1)
        P = torch.zeros((self.M, F.shape[1]), dtype=torch.complex128, device="cuda").index_add_(0, where, F)
        sup = torch.unique(where)
        return sup, P[sup] * self.sc[sup, None], torch.tensor(_delta(atom), device="cuda")

    def _axis(self, T, u, d):
        """Contract direction d (0 = x) of u [E, z, y, x, f] with T [in][out]."""
        return torch.matmul(T.T, u) if d == 0 else torch.matmul(
            T.T, u.reshape(u.shape[:3 - d] + (self.n, -1))).reshape(u.shape)

    def _chain(self, tabs, u):
        for d in range(3):
            u = self._axis(tabs[d], u, d)
        return u

    def local_fields(self, X):
        """The unscaled spinor at the quadrature points, [E][point][spin][col]."""
        n = X.shape[1]
        Z = torch.view_as_real((X.reshape(self.M, 2, n) * self.sc[:, None, None]).contiguous()).reshape(self.M, -1)
        u = Z[self.nodes].reshape(self.s.E, self.n, self.n, self.n, -1)
        U = self._chain((self.B,) * 3, u)
        return u, torch.view_as_complex(U.reshape(self.s.E, self.n ** 3, 2, n, 2).contiguous())

    def apply(self, X):
        step = max(1, int(6e8 // (self.s.E * self.n ** 3 * 4)))
        return torch.cat([self._apply(X[:, i:i + step].contiguous()) for i in range(0, X.shape[1], step)], 1)

    def _apply(self, X):
        s, n, E = self.s, X.shape[1], self.s.E
        u, U = self.local_fields(X)
        w = self.wJ[None, :, None]
        pot = self.V + 0.5 * sum(k * k for k in self.k)
        up, dn = U[:, :, 0], U[:, :, 1]
        bx, by, bz = (self.Bf[:, :, d, None] for d in range(3))
        W = torch.empty_like(U)
        W[:, :, 0] = w * ((pot[..., None] + bz) * up + torch.complex(bx, -by) * dn)
        W[:, :, 1] = w * ((pot[..., None] - bz) * dn + torch.complex(bx, by) * up)
        y = None
        shape = (E, self.n, self.n, self.n, -1)
        for d in range(3):
            tabs = [self.D if i == d else self.B for i in range(3)]
            g = self._chain(tabs, u).reshape(E, self.n ** 3, -1)
            if self.k[d]:
                G = torch.view_as_complex(g.reshape(E, self.n ** 3, 2, n, 2).contiguous())
                W -= 1j * self.k[d] * (w[..., None] * G)
            t = self._chain([m.T for m in tabs], (0.5 * w * g).reshape(shape))
            y = t if y is None else y.add_(t)
        y = y + self._chain([self.B.T] * 3, torch.view_as_real(W).reshape(shape))
        out = torch.zeros((self.M, 4 * n), dtype=torch.float64, device=X.device)
        out.index_add_(0, self.nodes.reshape(-1), y.reshape(E * self.n ** 3, -1))
        Y = torch.view_as_complex(out.reshape(self.M, 2, n, 2)) * self.sc[:, None, None]
        Xr = X.reshape(self.M, 2, n)
        for sup, P, delta in self.proj:
            c = (P.mH @ Xr[sup].reshape(len(sup), 2 * n)).reshape(-1, n)
            Y[sup] += (P @ (delta @ c).reshape(P.shape[1], 2 * n)).reshape(-1, 2, n)
        return Y.reshape(2 * self.M, n)

    def densities(self, X, f):
        """rho and m of occupations f, at the quadrature points."""
        rho, mag = 0.0, 0.0
        step = max(1, int(6e8 // (self.s.E * self.n ** 3 * 4)))
        for i in range(0, X.shape[1], step):
            r, b = _pair(*(self.local_fields(X[:, i:i + step].contiguous())[1],) * 2, f[i:i + step])
            rho, mag = rho + r, mag + b
        return rho, mag


def _pair(L, Y, f=None):
    """sum_n f_n l_n^H (1, sigma) y_n, real parts."""
    if f is not None:
        Y = Y * f
    lu, ld, yu, yd = L[:, :, 0].conj(), L[:, :, 1].conj(), Y[:, :, 0], Y[:, :, 1]
    uu, dd, ud, du = ((x * y).sum(-1) for x, y in ((lu, yu), (ld, yd), (lu, yd), (ld, yu)))
    return (uu + dd).real, torch.stack([(ud + du).real, (ud - du).imag, (uu - dd).real], -1)


def _coefficients(m, a, b, a0):
    """(alpha_k, beta_k), k = 1..m, and the shift of the scaled recurrence."""
    e, c = 0.5 * (b - a), 0.5 * (b + a)
    s1 = s = e / (a0 - c)
    al, be = [0.0, s1 / e], [0.0, 0.0]
    for _ in range(2, m + 1):
        t = 1.0 / (2.0 / s1 - s)
        al.append(2.0 * t / e)
        be.append(-s * t)
        s = t
    return al, be, c


def _filter(H, X, m, bounds, keep=False):
    al, be, c = _coefficients(m, *bounds)
    states, prev, Y = [X], None, X
    for k in range(1, m + 1):
        Z = al[k] * (H(Y) - c * Y)
        if k > 1:
            Z += be[k] * prev
        prev, Y = Y, Z
        if keep:
            states.append(Y)
    return states if keep else Y


def _fermi(theta, count):
    lo, hi = theta.min() - 60 * KT, theta.max() + 60 * KT
    for _ in range(200):
        mu = 0.5 * (lo + hi)
        x = np.clip((theta - mu) / KT, -700, 700)
        f = 1.0 / (1.0 + np.exp(x))
        lo, hi = (mu, hi) if f.sum() < count else (lo, mu)
    return f


def exact(case, seed):
    kind, n, m = case["kind"], case["vec"], case["degree"]
    if kind == "scf":
        return None                              # the loop's inner solves stop at a tolerance of their own
    s = System(case, seed)
    bounds = (A_CUT, s.bound(), A_LOW)
    if kind == "batch":
        out = []
        for t in range(case["tasks"]):
            y = System(case, 1000 * seed + t)
            out.append(_filter(Reference(y, *y.fields()).apply, y.random_block(1000 * seed + t, n), m, bounds))
        return torch.cat(out)
    if kind == "chol":
        return orthonormal(s.random_block(seed, n))
    ref = Reference(s, *s.fields())
    if kind in ("apply", "fields"):
        return ref.apply(s.random_block(seed, n))
    if kind == "filter":
        return _filter(ref.apply, s.random_block(seed, n), m, bounds)
    if kind == "resid":
        X, theta = s.smooth_block(seed, n)
        R = s.random_block(seed + 1, n).mul_(0.02)
        al, be, c = _coefficients(m, *bounds)
        th = torch.tensor(theta, device="cuda")
        p0, p1 = torch.ones_like(th), al[1] * (th - c)
        Z0, Z1 = torch.zeros_like(R), al[1] * R
        for k in range(2, m + 1):
            Z0, Z1 = Z1, al[k] * (ref.apply(Z1) - c * Z1) + be[k] * Z0 + R * (al[k] * p1)
            p0, p1 = p1, al[k] * (th - c) * p1 + be[k] * p0
        return X * p1 + Z1
    if kind == "ritz":
        X = orthonormal(s.smooth_block(seed, n)[0])
        W = ref.apply(X)
        theta, Q = torch.linalg.eigh((X.mH @ W).cpu())
        Q = Q.to(X.device)
        X, W = X @ Q, W @ Q
        resid = (W - X * theta.to(X.device)).norm(dim=0)
        occ = _fermi(theta.numpy(), 0.8 * n)
        rho, mag = ref.densities(X, torch.tensor(occ, device=X.device))
        return theta, resid, occ, rho, mag
    if kind == "lanczos":
        v = s.random_block(seed, 1)
        v, prev, beta, al, be = v / v.norm(), torch.zeros_like(v), 0.0, [], []
        for _ in range(m):
            w = ref.apply(v)
            alpha = float((v.conj() * w).real.sum())
            w = w - alpha * v - beta * prev
            beta = float(w.norm())
            al.append(alpha)
            be.append(beta)
            prev, v = v, w / beta
        t = np.linalg.eigvalsh(np.diag(al) + np.diag(be[:-1], 1) + np.diag(be[:-1], -1))
        return float(t[0]), float(t[-1] + be[-1])
    if kind == "adjoint":
        al, be, c = _coefficients(m, *bounds)
        Y = _filter(ref.apply, s.random_block(seed, n), m, bounds, keep=True)
        lam, nxt, dV, dB = s.random_block(seed + 2, n), None, 0.0, 0.0
        for k in range(m, 0, -1):
            r, b = _pair(ref.local_fields(lam)[1], ref.local_fields(Y[k - 1])[1])
            dV, dB = dV + al[k] * r * ref.wJ, dB + al[k] * b * ref.wJ[:, None]
            t = al[k] * (ref.apply(lam) - c * lam)
            lam, nxt = (t if nxt is None else t + be[k + 1] * nxt), lam
        return Y[-1], lam, dV, dB
    raise KeyError(kind)
