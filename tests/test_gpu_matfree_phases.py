"""The matrix-free product at every order, at Gamma and at a k-point, in both precisions:
its x pass runs the spins together or one by one, and the fields are padded in LDS at
n_p = 8, depending on all three.  Against the stored cell matrices to 1e-12 of the
largest value in FP64, and within 2e-6 of them in FP32 (the bounds of the parity tests
of the form); the filter by colours and by cells bit for bit."""
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _op(p, k, form):
    from paper_2410_02754_amd import Operator
    s = synth.make_system("phases", n_cells=(3, 2, 2), box=(3.3, 2.4, 2.0), p=p, kpts=[(k, -k, 0.5 * k)], n_atoms=1,
                          lmax=1, rcut_sigmas=4.0, n_vec=1, b_mag=0.7, b_bias=(0.3, -0.4, 0.5))
    op = Operator(s.n_cells, s.box, s.p, s.quad, s.n_q, s.kpts, form=form)
    pts = op.quad_points().reshape(-1, 3)
    op.set_local(torch.tensor(synth.veff(s, pts).reshape(op.n_cells, op.nq3), device="cuda"),
                 torch.tensor(synth.bxc(s, pts).reshape(op.n_cells, op.nq3, 3), device="cuda"))
    op.set_atoms(s.atoms)
    return op


@pytest.mark.parametrize("k", [0.0, 0.3])
@pytest.mark.parametrize("p", range(1, 9))
def test_every_order_matches_cell_matrices(p, k):
    mf, cell = _op(p, k, "matrix_free"), _op(p, k, "cell")
    X = torch.tensor(synth.random_block(p, mf.n_dof, 19), device="cuda")
    ref = cell.apply_H(X, torch.empty_like(X))
    for prec, low, tol in (("fp64", 0.0, 1e-12), ("mixed", 1e-9, 2e-6)):
        Y = mf.apply_H(X, torch.empty_like(X), prec=prec)
        err = float((Y - ref).abs().max() / ref.abs().max())
        assert low <= err < tol, (prec, err)
        W, A, B = torch.empty_like(X), X.clone(), X.clone()
        mf.cheb_filter(A, W, 3, 8.0, 900.0, -6.0, prec=prec)
        mf.cheb_filter_noalloc(B, W, 3, 8.0, 900.0, -6.0, prec=prec)
        assert torch.isfinite(torch.view_as_real(A)).all() and torch.equal(A, B)
    mf.close()
    cell.close()
