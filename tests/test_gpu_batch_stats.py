"""Stage statistics of a batch run by plain launches: small tasks, which go together, are
counted per context as the per-task filters of the same blocks are (the counts to
rounding), and their time is recorded."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _op(cells, p, k, lmax, form, stream):
    from paper_2410_02754_amd import Operator
    s = synth.make_system("stats", n_cells=cells, box=tuple(1.2 * c for c in cells), p=p, kpts=[(k, -k, 0.5 * k)],
                          n_atoms=2, lmax=lmax, rcut_sigmas=4.0, n_vec=1)
    op = Operator(s.n_cells, s.box, s.p, s.quad, s.n_q, s.kpts, stream=stream.cuda_stream, form=form)
    pts = op.quad_points().reshape(-1, 3)
    op.set_local(torch.tensor(synth.veff(s, pts).reshape(op.n_cells, op.nq3), device="cuda"),
                 torch.tensor(synth.bxc(s, pts).reshape(op.n_cells, op.nq3, 3), device="cuda"))
    op.set_atoms(s.atoms)
    return op


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_small_tasks_are_counted_per_context(prec):
    from paper_2410_02754_amd.chfsi import Batch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ops = [_op((3, 2, 2), 4, 0.2, 1, "cell", stream), _op((2, 3, 3), 3, 0.0, 2, "matrix_free", stream)]
        tasks = []
        for op, n in ((ops[0], 12), (ops[1], 20), (ops[0], 7)):
            X = torch.tensor(synth.random_block(n, op.n_dof, n), device="cuda")
            tasks.append((op, 0, X, torch.empty_like(X)))
        batch = Batch(tasks, 5, prec=prec, flags=0)
        got, want = [], []
        for run, out in ((lambda: batch.filter(8.0, 900.0, -6.0), got),
                         (lambda: [op.cheb_filter(X, W, 5, 8.0, 900.0, -6.0, prec=prec) for op, _, X, W in tasks], want)):
            for op in ops:
                op.stats_reset()
                op.stats_enable(True)
            run()
            torch.cuda.synchronize()
            for op in ops:
                out.append(op.stats())
                op.stats_enable(False)
        for a, b in zip(got, want):
            for stage in ("nonlocal", "axpy"):
                assert a[stage]["ms"] > 0.0 and a[stage]["launches"] > 0
                for what in ("flops", "bytes"):
                    assert np.isclose(a[stage][what], b[stage][what], rtol=1e-12, atol=0.0), (stage, what)
        batch.close()
        for op in ops:
            op.close()
