"""Step limits of the field solves, around the sixteen steps between the host's looks: a
limit below the converged count is reported as a negative count of that many steps, the
converged count itself and any larger limit as the count."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("cells,p", [((3, 4, 5), 4), ((9, 8, 7), 1), ((4, 5, 3), 2)])
def test_counts_at_step_limits(cells, p):
    from paper_2410_02754_amd import Operator
    op = Operator(cells, tuple(1.3 * c for c in cells), p, "gl", p + 1)
    rng = np.random.default_rng(5)
    r = torch.tensor(rng.uniform(0.1, 1.0, (op.n_cells, op.nq3)), device="cuda")
    out, ref = torch.empty_like(r), torch.empty_like(r)
    for solve in (lambda o, m: op.hartree(r, o, tol=1e-12, max_iter=m),
                  lambda o, m: op.kerker(r, o, 0.3, tol=1e-12, max_iter=m)):
        n = solve(ref, 5000)
        assert n > 18
        for m in (1, 2, 15, 16, 17, n - 1):
            assert solve(out, m) == -m
        for m in (n, n + 1, n + 40):
            out.zero_()
            assert solve(out, m) == n and torch.equal(out, ref)
    op.close()
