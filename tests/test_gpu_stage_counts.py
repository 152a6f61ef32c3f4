"""Counts of the stage statistics against the work of the kernels that run: the
matrix-free product makes 9 line contractions per spin in FP64 at Gamma and 12
otherwise (8 n_p^4 flops each, two spins), the cell kernel issues MFMAs for the waves that
have a column, and the gather of the cells' products is counted in bytes."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _counts(p, k, form, n, prec):
    from paper_2410_02754_amd import Operator
    op = Operator((3, 2, 2), (3.6, 2.4, 2.4), p, "gl", p + 1, [(k, 0.0, 0.0)], form=form)
    V = torch.rand((op.n_cells, op.nq3), dtype=torch.float64, device="cuda")
    B = torch.rand((op.n_cells, op.nq3, 3), dtype=torch.float64, device="cuda")
    op.set_local(V, B)
    X = torch.randn((op.n_dof, n), dtype=torch.complex128, device="cuda")
    op.stats_enable(True)
    op.apply_H(X, torch.empty_like(X), prec=prec)
    st = op.stats()
    rows, cells = op.n_dof, op.n_cells
    op.close()
    gather = 2 * cells * (p + 1)**3 * n * (8 if prec == "mixed" else 16)
    assert st["axpy"]["bytes"] == rows * n * 16 + gather      # alone: no recurrence terms
    return st["cell_fp32" if prec == "mixed" else "cell_fp64"]["exec_flops"], cells


@pytest.mark.parametrize("k,prec,lines", [(0.0, "fp64", 9), (0.2, "fp64", 12), (0.0, "mixed", 12)])
def test_line_contractions(k, prec, lines):
    got, cells = _counts(4, k, "matrix_free", 10, prec)
    assert got == lines * 2 * 4 * 5**4 * 10 * cells           # complex by real: 4 flops a multiply-add


@pytest.mark.parametrize("prec,n,blocks", [("fp64", 130, 9), ("mixed", 130, 10), ("fp64", 20, 2), ("mixed", 64, 4)])
def test_cell_kernel_column_blocks(prec, n, blocks):
    got, cells = _counts(3, 0.0, "cell", n, prec)
    nloc = 64
    assert got == cells * (nloc // 16) * blocks * (nloc // 4) * 8 * 2048
