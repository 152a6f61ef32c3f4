"""Hartree and Kerker solves at every order of basis, with two cells in a direction
(a node's frame then holds the same node on both sides), odd counts and quadratures
other than p + 1, against the oracle's direct solve.  Tolerance as in the other
parity tests of the solves: 1e-11 relative (CG to 1e-13 on operators of condition
number below 1e3 after scaling)."""
import numpy as np
import pytest

from oracle import fe, scf

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("p,nq,nc", [(1, 2, (2, 3, 4)), (2, 3, (2, 2, 5)), (3, 6, (3, 2, 2)), (4, 5, (2, 3, 3)),
                                     (5, 6, (2, 2, 2)), (6, 9, (2, 2, 2)), (7, 8, (2, 2, 2)), (8, 9, (2, 2, 2))])
def test_solves_match_oracle(p, nq, nc):
    from paper_2410_02754_amd import Operator
    box = tuple(1.7 * n for n in nc)
    m = fe.Mesh(nc, box, p, "gl", nq)
    op = Operator(nc, box, p, "gl", nq)
    pts = m.all_quad_points()
    rho = 0.1 + np.exp(-np.sum((pts - 0.4 * np.array(box)) ** 2, axis=-1)) + 0.05 * np.cos(
        2 * np.pi * pts[..., 0] / box[0])
    r = torch.tensor(rho, device="cuda")
    out = torch.empty_like(r)
    assert op.hartree(r, out) > 0
    ref = scf.hartree(m, rho)
    assert np.abs(out.cpu().numpy() - ref).max() < 1e-11 * np.abs(ref).max()
    assert op.kerker(r, out, 0.8) > 0
    ref = scf.kerker(m, rho, 0.8)
    assert np.abs(out.cpu().numpy() - ref).max() < 1e-11 * np.abs(ref).max()
    # a step limit that is not reached in time is reported as a negative count
    assert op.hartree(r, out, max_iter=1) in (1, -1)
    z = torch.zeros_like(r)
    assert op.hartree(z, out) == 0 and float(out.abs().max()) == 0.0
    op.close()
