"""chfsi_workspace_bytes of one call on a fresh context against the device memory it
takes: a Rayleigh-Ritz step whose Gram sums are larger than the applies' coefficients,
and a mixed filter whose single-precision applies keep the cells' products while the
double-precision one does not.  8 MiB for the allocator's rounding."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _op(cells, p, form, n):
    from paper_2410_02754_amd import Operator
    op = Operator((cells,) * 3, (1.2 * cells,) * 3, p, "gl", p + 1, form=form)
    V = torch.rand((op.n_cells, op.nq3), dtype=torch.float64, device="cuda")
    B = torch.rand((op.n_cells, op.nq3, 3), dtype=torch.float64, device="cuda")
    op.set_local(V, B)
    X = torch.zeros((op.n_dof, n), dtype=torch.complex128, device="cuda")
    X[:2 * n:2] = torch.eye(n, dtype=torch.complex128, device="cuda")      # orthonormal columns
    W = torch.empty_like(X)
    torch.cuda.synchronize()
    return op, X, W


def _taken(f):
    free = torch.cuda.mem_get_info()[0]
    f()
    torch.cuda.synchronize()
    return free - torch.cuda.mem_get_info()[0]


def test_rayleigh_ritz_counts_products_and_gram_sums():
    op, X, W = _op(6, 4, "cell", 64)
    bound = op.workspace_bytes(64, "rayleigh_ritz")
    used = _taken(lambda: op.rayleigh_ritz(X, W))
    assert op.workspace_bytes(64, "apply") < used <= bound + (8 << 20), (used, bound)
    op.close()


@pytest.mark.parametrize("n", [72, 16])
def test_filter_counts_either_precision(n):
    # 20^3 cells, p = 2: 8 columns a workgroup in FP64, 16 in FP32; at 72 columns only the
    # FP32 products go cell by cell
    op, X, W = _op(20, 2, "matrix_free", n)
    bound = op.workspace_bytes(n, "filter")
    used = _taken(lambda: op.cheb_filter(X, W, 3, 8.0, 900.0, -6.0, prec="mixed"))
    assert 8000 * 27 * 2 * n * 8 <= used + (8 << 20) and used <= bound + (8 << 20), (used, bound)
    op.close()
