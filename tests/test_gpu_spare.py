"""Many contexts whose products each want 1.4 GB for the cells' values: together they hold
at most 8 GiB of it, and those without it give the same bits by colours."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def test_many_contexts_share_a_bound():
    from paper_2410_02754_amd import Operator
    n, made = 256, []
    g = torch.Generator(device="cuda").manual_seed(1)
    for i in range(8):
        op = Operator((8, 8, 8), (9.6, 9.6, 9.6), 6, "gl", 7, form="matrix_free")
        if i == 0:
            V = torch.rand((op.n_cells, op.nq3), dtype=torch.float64, device="cuda", generator=g)
            B = torch.rand((op.n_cells, op.nq3, 3), dtype=torch.float64, device="cuda", generator=g)
            X = torch.randn((op.n_dof, n), dtype=torch.complex128, device="cuda", generator=g)
            Y = torch.empty_like(X)
        op.set_local(V, B)
        made.append(op)
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    want = None
    for op in made:
        Y.zero_()
        op.apply_H(X, Y)
        op.apply_H(X, Y)
        torch.cuda.synchronize()
        if want is None:
            want = Y.clone()
            free0 -= want.numel() * 16
        assert torch.equal(Y, want)
    held = free0 - torch.cuda.mem_get_info()[0]
    each = made[0].n_cells * 343 * 2 * n * 16
    assert each < held < (8 << 30) + (64 << 20), held
    for op in made:
        op.close()
    torch.cuda.synchronize()
    assert free0 - torch.cuda.mem_get_info()[0] < (64 << 20)
