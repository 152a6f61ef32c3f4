"""Cell operators at every order of basis and at the edges of their blocks: the
dense cell product (stored matrices) against the matrix-free product, which
shares none of the setup, and, for quadratures that only the stored form takes,
against the oracle.  Tolerance: both are sums of at most (p + 1)^3 (n_q)^3 terms of one
operator in FP64; 1e-12 relative as in the other parity tests of the apply."""
import numpy as np
import pytest

import synth
from oracle import hamiltonian as ham

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _system(p, n_q=None, k=(0.1, -0.2, 0.15), cells=(2, 3, 2)):
    return synth.make_system("setup", n_cells=cells, box=tuple(1.5 * c for c in cells), p=p, n_q=n_q, kpts=[k],
                             n_atoms=1, lmax=0, rcut_sigmas=3.0, n_vec=5, b_mag=0.4)


def _op(s, form):
    from paper_2410_02754_amd import Operator
    op = Operator(s.n_cells, s.box, s.p, s.quad, s.n_q, s.kpts, form=form)
    pts = op.quad_points().reshape(-1, 3)
    op.set_local(torch.tensor(synth.veff(s, pts).reshape(op.n_cells, op.nq3), device="cuda"),
                 torch.tensor(synth.bxc(s, pts).reshape(op.n_cells, op.nq3, 3), device="cuda"))
    return op


@pytest.mark.parametrize("p", range(1, 9))
@pytest.mark.parametrize("k", [(0.0, 0.0, 0.0), (0.1, -0.2, 0.15)])
def test_stored_matrices_equal_matrix_free(p, k):
    s = _system(p, k=k)
    ops = [_op(s, f) for f in ("cell", "matrix_free")]
    X = torch.tensor(synth.start_block(s, s.n_dof), device="cuda")
    Y = [op.apply_H(X, torch.empty_like(X)) for op in ops]
    err = float((Y[0] - Y[1]).abs().max() / Y[1].abs().max())
    assert err < 1e-12, err
    for op in ops:
        op.close()


@pytest.mark.parametrize("p,n_q", [(2, 2), (3, 6), (4, 9), (8, 12)])
def test_other_quadratures_match_oracle(p, n_q):
    cells = (2, 2, 2) if p < 8 else (2, 2, 2)
    s = _system(p, n_q, cells=cells)
    op = _op(s, "cell")
    X0 = synth.start_block(s, s.n_dof)
    X = torch.tensor(X0, device="cuda")
    Y = op.apply_H(X, torch.empty_like(X)).cpu().numpy()
    mesh, H, _, _, _ = ham.build(s, synth.veff, synth.bxc, atoms=[])
    ref = H @ X0
    assert np.abs(Y - ref).max() < 1e-12 * np.abs(ref).max()
    op.close()
