"""Field solves on meshes with more nodes or cells than one round of workgroups takes: a
thread per node (orders 1 and 2) and a workgroup per cell, several parts per thread of
the sums.  With Gauss-Lobatto quadrature of p + 1 points the points are the nodes, so the
Kerker output gives the nodal solution, whose residual is formed here in 64 bits.

Tolerance: the solve stops at a recursive residual of 1e-13 of the right-hand side; the
true one differs by roundings of |A| |u| <= cond |b| (below 1e3) times a few eps, so
1e-11 as in the parity tests of the solves."""
import numpy as np
import pytest

from oracle import fe, scf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

H, K0 = 1.7, 0.8


def _nodes(nc, p):
    """Global node of each quadrature point, [E][(p + 1)^3], in the library's orders."""
    n = [c * p for c in nc]
    q = np.arange(p + 1)
    ax = [((np.arange(c)[:, None] * p + q) % m) for c, m in zip(nc, n)]
    x = ax[0][None, None, :, None, None, :]
    y = ax[1][None, :, None, None, :, None]
    z = ax[2][:, None, None, :, None, None]
    return (x + n[0] * (y + n[1] * z)).reshape(np.prod(nc), -1)


def _solve(nc, p, rho):
    """(k0^2 - lap)^{-1} rho at the nodes, from the Kerker filter of rho."""
    from paper_2410_02754_amd import Operator
    op = Operator(nc, tuple(H * c for c in nc), p, "gll", p + 1)
    idx = _nodes(nc, p)
    r = torch.tensor(rho[idx], device="cuda")
    out = torch.empty_like(r)
    assert op.kerker(r, out, K0) > 0
    w = ((r - out) / K0**2).cpu().numpy()
    op.close()
    u = np.empty(rho.size)
    u[idx.ravel()] = w.ravel()
    return u, idx


def test_order_one_more_nodes_than_threads():
    nc = (83, 81, 82)                    # 551286 nodes, 524288 threads at most
    rho = np.random.default_rng(3).uniform(-1, 1, int(np.prod(nc)))
    u, _ = _solve(nc, 1, rho)
    # h M = h I, S = [-1, 2, -1] / h: diagonal in the Fourier basis
    lam = [(2 - 2 * np.cos(2 * np.pi * np.arange(n) / n)) / H**2 for n in nc]
    sym = K0**2 + lam[2][:, None, None] + lam[1][None, :, None] + lam[0][None, None, :]
    v = u.reshape(nc[2], nc[1], nc[0])
    Au = np.fft.ifftn(np.fft.fftn(v) * sym).real.ravel()
    assert np.linalg.norm(Au - rho) < 1e-11 * np.linalg.norm(rho)


@pytest.mark.parametrize("p,nc", [(2, (20, 21, 22)), (2, (2, 3, 2)), (3, (13, 14, 13)), (4, (7, 9, 8))])
def test_residual_of_the_nodal_solution(p, nc):
    rho = np.random.default_rng(4).uniform(-1, 1, int(np.prod(nc)) * p**3)
    u, idx = _solve(nc, p, rho)
    m = fe.Mesh(nc, tuple(H * c for c in nc), p, "gll", p + 1)
    b = scf.project(m, rho[idx])
    r = b - scf.scalar_operator(m, K0**2) @ u
    assert np.linalg.norm(r) < 1e-11 * np.linalg.norm(b)


@pytest.mark.parametrize("p,nc", [(1, (64, 32, 32)), (1, (65, 32, 32)), (3, (8, 8, 4)), (3, (43, 3, 2))])
def test_around_256_parts(p, nc):
    """256 parts of the sums and a few more, by nodes and by cells."""
    test_residual_of_the_nodal_solution(p, nc)
