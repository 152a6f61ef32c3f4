"""Whole Gram products with tiles of 64 and of 128 rows (from 512 columns on, by how the
tiles fill the columns and the GPU), ragged last tiles, in wider arrays, against
complex128 products.  Tolerance as in the tests of the smaller tiles."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cells,p", [((2, 2, 2), 1), ((3, 3, 2), 3), ((19, 14, 26), 1)])
@pytest.mark.parametrize("n", [448, 511, 512, 576, 577, 640, 900])
def test_whole_product(cells, p, n):
    from paper_2410_02754_amd import Operator
    op = Operator(cells, tuple(1.1 * c for c in cells), p, "gll", p + 1)
    A = torch.tensor(synth.random_block(1, op.n_dof, n + 5), device="cuda")
    x, y = A[:, :n], torch.tensor(synth.random_block(2, op.n_dof, n), device="cuda")
    want = (x.conj().T.contiguous() @ y).cpu().numpy()
    scale = np.sqrt(np.outer((x.abs()**2).sum(0).cpu().numpy(), (y.abs()**2).sum(0).cpu().numpy()))
    assert np.max(np.abs(op.overlap(x, y) - want) / scale) < 1e-12
    op.close()
