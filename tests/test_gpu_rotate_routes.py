"""Triangular rotations on both sides of the row counts at which they go from panels to
in place (128 tiles of 64 rows up to 128 columns, 216 above), last row and column tiles
full and ragged, in a wider array, against complex128 products.

Tolerance as in the tests of the tiles: sums of at most 14000 terms of unit columns."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cells,p,tiles", [((16, 16, 16), 1, 128), ((16, 16, 17), 1, 136), ((12, 9, 8), 2, 216),
                                           ((19, 14, 26), 1, 217), ((3, 3, 2), 3, 16)])
@pytest.mark.parametrize("n", [64, 65, 128, 129, 200])
def test_triangular_rotation(cells, p, tiles, n):
    from paper_2410_02754_amd import Operator
    op = Operator(cells, tuple(1.1 * c for c in cells), p, "gll", p + 1)
    rows = op.n_dof
    assert -(-rows // 64) == tiles
    X = torch.full((rows, n + 3), 7.0, dtype=torch.complex128, device="cuda")
    X[:, :n] = torch.tensor(synth.random_block(n, rows, n), device="cuda")
    x = X[:, :n]
    xc = x.contiguous()
    L = np.linalg.cholesky((xc.conj().T.contiguous() @ xc).cpu().numpy())
    ref = xc @ torch.tensor(np.ascontiguousarray(np.linalg.inv(L).conj().T), device="cuda")
    op.chol_gs(x)
    torch.cuda.synchronize()
    assert torch.max((x - ref).abs()) < 1e-12 * torch.max(ref.abs())
    assert (X[:, n:] == 7.0).all()
    op.close()
