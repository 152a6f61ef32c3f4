"""Small tasks of a batch share one launch per stage of a step: against the
per-task filter, bit for bit, with more tasks than one cell launch takes, with and
without atoms, real, packed and unpacked projectors, both forms, and one task too
large to join them; by launches and as a graph replayed for new bounds."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

#        cells, p, lmax (None: no atoms), k, columns, form
KINDS = [((2, 2, 2), 3, 1, 0.2, 5, "cell"),
         ((3, 2, 2), 4, 2, 0.2, 70, "cell"),
         ((2, 3, 3), 2, 2, 0.0, 33, "cell"),
         ((2, 2, 3), 5, None, 0.1, 1, "cell"),
         ((3, 3, 2), 3, 1, 0.1, 20, "matrix_free"),
         ((2, 2, 2), 6, 2, 0.0, 130, "matrix_free"),
         ((2, 2, 2), 4, 2, 0.1, 1, "cell"),
         ((2, 3, 2), 3, 1, 0.0, 1, "matrix_free")]
LARGE = ((41, 41, 41), 1, 0, 0.0, 2, "cell")     # 68921 workgroups in eight colours


def _op(kind, stream):
    from paper_2410_02754_amd import Operator
    cells, p, lmax, k, _, form = kind
    s = synth.make_system("small", n_cells=cells, box=tuple(1.2 * c for c in cells), p=p, kpts=[(k, -k, 0.5 * k)],
                          n_atoms=2, lmax=lmax or 0, rcut_sigmas=4.0, n_vec=1)
    op = Operator(s.n_cells, s.box, s.p, s.quad, s.n_q, s.kpts, stream=stream.cuda_stream, form=form)
    pts = op.quad_points().reshape(-1, 3)
    op.set_local(torch.tensor(synth.veff(s, pts).reshape(op.n_cells, op.nq3), device="cuda"),
                 torch.tensor(synth.bxc(s, pts).reshape(op.n_cells, op.nq3, 3), device="cuda"))
    if lmax is not None:
        op.set_atoms(s.atoms)
    return op


@pytest.mark.parametrize("prec,degree,graph,large", [("fp64", 3, True, True), ("mixed", 4, True, False),
                                                     ("mixed", 1, False, True), ("fp64", 2, False, False)])
def test_small_tasks_equal_per_task_bitwise(prec, degree, graph, large):
    from paper_2410_02754_amd.chfsi import BATCH_GRAPH, Batch
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        kinds = KINDS + ([LARGE] if large else [])
        ops = [_op(k, stream) for k in kinds]
        tasks = []
        for t in range(5 * len(KINDS) + (1 if large else 0)):       # more than 32
            j = t % len(KINDS) if t < 5 * len(KINDS) else len(KINDS)
            X = torch.tensor(synth.random_block(t, ops[j].n_dof, kinds[j][4]), device="cuda")
            tasks.append((ops[j], 0, X, torch.empty_like(X)))
        X0 = [t[2].clone() for t in tasks]
        batch = Batch(tasks, degree, prec=prec, flags=BATCH_GRAPH if graph else 0)
        for rep in range(3):
            a = np.array([8.0 + rep + 0.1 * t for t in range(len(tasks))])
            b, a0 = a + 900.0, a - 15.0
            for (_, _, X, _), x0 in zip(tasks, X0):
                X.copy_(x0)
            batch.filter(a, b, a0)
            torch.cuda.synchronize()
            for t, (op, _, X, _) in enumerate(tasks):
                Y = X0[t].clone()
                op.cheb_filter(Y, torch.empty_like(Y), degree, a[t], b[t], a0[t], prec=prec)
                torch.cuda.synchronize()
                assert torch.isfinite(torch.view_as_real(X)).all()
                assert torch.equal(Y, X), f"task {t}, pass {rep}"
        batch.close()
        for op in ops:
            op.close()
