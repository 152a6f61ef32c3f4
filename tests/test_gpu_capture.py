"""A product captured by the caller into a graph: replays after later, wider products on
the same context (which move its own buffers) give the eager result.  Operators without
atoms, which allocate nothing that a graph would have to keep; both forms, and both
kinds of capture (before and after the first eager product)."""
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("form,k,prec,first", [("cell", 0.0, "fp64", True), ("matrix_free", 0.2, "mixed", True),
                                               ("matrix_free", 0.0, "fp64", False)])
def test_captured_product_survives_wider_ones(form, k, prec, first):
    from paper_2410_02754_amd import Operator
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        op = Operator((3, 4, 3), (3.6, 4.8, 3.6), 4, "gl", 5, [(k, 0.0, -k)], stream=stream.cuda_stream, form=form)
        V = torch.rand((op.n_cells, op.nq3), dtype=torch.float64, device="cuda")
        B = torch.rand((op.n_cells, op.nq3, 3), dtype=torch.float64, device="cuda")
        op.set_local(V, B)
        X = torch.tensor(synth.random_block(1, op.n_dof, 8), device="cuda")
        Y = torch.zeros_like(X)
        if first:
            op.apply_H(X, Y, prec=prec)
        stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        op.apply_H(X, Y, prec=prec)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        for n in (8, 40, 160, 16):
            W = torch.tensor(synth.random_block(n, op.n_dof, n), device="cuda")
            Z = op.apply_H(W, torch.empty_like(W), prec=prec)
            fill = torch.full((1 << 22,), float("nan"), dtype=torch.float64, device="cuda")   # takes freed memory
            X.copy_(W[:, :8])
            Y.zero_()
            g.replay()
            torch.cuda.synchronize()
            want = op.apply_H(X, torch.empty_like(X), prec=prec)
            torch.cuda.synchronize()
            assert torch.equal(Y, want), n
            del fill, Z
    op.close()


def test_captured_narrower_block_after_a_wider_warm_up():
    """With atoms the scratch cannot grow under capture: what a wide product has taken serves
    every narrower one, whose sums are cut into more parts."""
    from paper_2410_02754_amd import Operator
    s = synth.make_system("many", n_cells=(4, 4, 4), box=(4.0, 4.0, 4.0), p=6, n_atoms=40, lmax=1, rcut_sigmas=8.0,
                          n_vec=1)
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        op = Operator(s.n_cells, s.box, s.p, s.quad, s.n_q, s.kpts, stream=stream.cuda_stream, form="matrix_free")
        op.set_local(torch.rand((op.n_cells, op.nq3), dtype=torch.float64, device="cuda"),
                     torch.rand((op.n_cells, op.nq3, 3), dtype=torch.float64, device="cuda"))
        op.set_atoms(s.atoms)
        W = torch.tensor(synth.random_block(1, op.n_dof, 144), device="cuda")
        op.apply_H(W, torch.empty_like(W))
        widths = {n: W[:, :n].contiguous() for n in (3, 16, 64, 100)}
        out = {n: torch.zeros_like(x) for n, x in widths.items()}
        stream.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream, capture_error_mode="thread_local"):
        for n, x in widths.items():
            op.apply_H(x, out[n])
    torch.cuda.synchronize()
    for rep in range(3):
        with torch.cuda.stream(stream):
            for n, x in widths.items():
                x.mul_(1.5)
                out[n].zero_()
            g.replay()
            torch.cuda.synchronize()
            for n, x in widths.items():
                want = op.apply_H(x, torch.empty_like(x))
                torch.cuda.synchronize()
                assert torch.equal(out[n], want), n
    op.close()
