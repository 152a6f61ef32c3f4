"""Gram products and triangular rotations at the edges of their 64-wide tiles, with
ldx > n, below and above the row count from which the rotation goes in place,
against complex128 products of the same blocks.

Tolerance: sums of at most 72000 terms of unit columns; random-walk growth of their
rounding is sqrt(72000) eps = 6e-14 of a column's scale, and the blocks are close to
orthogonal, so the factor does not enlarge it: 1e-12 leaves a factor of ten and more."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _gram_loss(op, X):
    n = X.shape[1]
    return np.max(np.abs(op.overlap(X, X) - np.eye(n)))


def _block(rows, n, pad, seed):
    X = torch.zeros((rows, n + pad), dtype=torch.complex128, device="cuda")
    X[:, :n] = torch.tensor(synth.random_block(seed, rows, n), device="cuda")
    return X


@pytest.mark.parametrize("cells,p", [((3, 3, 3), 2), ((33, 33, 33), 1)])
@pytest.mark.parametrize("n,pad", [(1, 0), (31, 3), (64, 0), (65, 7), (130, 0), (193, 1)])
def test_gram_and_triangular_rotation(cells, p, n, pad):
    from paper_2410_02754_amd import Operator
    op = Operator(cells, tuple(1.1 * c for c in cells), p, "gll", p + 1, [(0.0, 0.0, 0.0)])
    rows = op.n_dof
    X, Y = _block(rows, n, pad, 1), _block(rows, n, pad, 2)
    x, y = X[:, :n], Y[:, :n]
    S = op.overlap(x, y)
    want = (x.conj().T.contiguous() @ y.contiguous()).cpu().numpy()
    scale = np.sqrt(np.outer((x.abs()**2).sum(0).cpu().numpy(), (y.abs()**2).sum(0).cpu().numpy()))
    assert np.max(np.abs(np.asarray(S) - want) / scale) < 1e-12
    xc = x.contiguous()
    L = np.linalg.cholesky((xc.conj().T.contiguous() @ xc).cpu().numpy())
    ref = xc @ torch.tensor(np.ascontiguousarray(np.linalg.inv(L).conj().T), device="cuda")
    op.chol_gs(x)
    torch.cuda.synchronize()
    assert torch.max((x - ref).abs()) < 1e-12 * torch.max(ref.abs())
    assert pad == 0 or torch.equal(X[:, n:], torch.zeros_like(X[:, n:]))
    op.close()


@pytest.mark.parametrize("n,dup", [(2, (0, 1)), (40, (3, 31)), (33, (0, 32)), (96, (70, 95))])
def test_failed_pivot_and_bad_values(n, dup):
    """A zero column, a NaN and a column of only its predecessors are refused, with the
    column named, and the block stays as it was."""
    from paper_2410_02754_amd import ChfsiError, Operator
    op = Operator((4, 3, 3), (4.4, 3.3, 3.3), 3, "gll", 4, [(0.0, 0.0, 0.0)])
    X0 = _block(op.n_dof, n, 0, 5)
    X = X0.clone()
    op.chol_gs(X)
    assert _gram_loss(op, X) < 1e-13
    for what, col in (("zero", dup[1]), ("nan", -1), ("huge", None)):
        X = X0.clone()
        if what == "zero":
            X[:, dup[1]] = 0.0
        elif what == "nan":
            X[5, dup[0]] = complex("nan")
        else:                                       # columns of very different norms are not an error
            X[:, dup[1]] *= 1e100
            X[:, dup[0]] *= 1e-100
            op.chol_gs(X)
            assert _gram_loss(op, X) < 1e-13
            continue
        Y = X.clone()
        with pytest.raises(ChfsiError) as e:
            op.chol_gs(X)
        assert e.value.bad_col == col
        assert torch.equal(torch.view_as_real(X).nan_to_num(7.0), torch.view_as_real(Y).nan_to_num(7.0))
    op.close()


@pytest.mark.parametrize("n", [1, 2, 3, 40, 41, 133])
def test_rayleigh_ritz_against_dense_eigenvalues(n):
    """One thread (n <= 40) and several, widths beside multiples of eight: Ritz values
    against numpy's of the same projected matrix, and the rotated block's projection
    diagonal, both to n^(3/2) roundings of the matrix' norm."""
    from paper_2410_02754_amd import Operator
    s = synth.make_system("rr", n_cells=(4, 3, 3), box=(4.8, 3.6, 3.6), p=3, kpts=[(0.1, 0.2, 0.0)], n_atoms=1, lmax=1,
                          rcut_sigmas=4.0, n_vec=1)
    op = Operator(s.n_cells, s.box, s.p, s.quad, s.n_q, s.kpts)
    pts = op.quad_points().reshape(-1, 3)
    op.set_local(torch.tensor(synth.veff(s, pts).reshape(op.n_cells, op.nq3), device="cuda"),
                 torch.tensor(synth.bxc(s, pts).reshape(op.n_cells, op.nq3, 3), device="cuda"))
    op.set_atoms(s.atoms)
    X = _block(op.n_dof, n, 0, 11)
    op.chol_gs(X)
    W = torch.empty_like(X)
    H = op.overlap(X, op.apply_H(X, W))
    want = np.linalg.eigvalsh((H + H.conj().T) / 2)
    theta, _ = op.rayleigh_ritz(X, W)
    tol = 4 * max(n, 4)**1.5 * np.finfo(float).eps * np.abs(want).max()
    assert np.max(np.abs(np.asarray(theta) - want)) < tol
    G = op.overlap(X, op.apply_H(X, W))
    assert np.max(np.abs(G - np.diag(np.asarray(theta)))) < 4 * tol
    op.close()
