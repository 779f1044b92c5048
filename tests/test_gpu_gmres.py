"""GMRES at the edges of its iteration: vectors of less than one block up to more than the 128 blocks
that sum a dot product's partials in the kernels that use them, restarts every few iterations,
iteration limits in the middle of a cycle and right after a queued iteration, and solves in a row on
the same context (the same to the bit).

The residual |b - A x| / |b| is recomputed from the operator's own product: at most the tolerance plus
1e-13 (rounding of one product); iteration counts stay within the limit given."""

import numpy as np
import pytest

from workloads import coax_problem, floating_shell_problem, sphere_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_12663_amd as bem
    return bem


def _residual(c, p, sol):
    b = c.rhs(p.body_V)
    r = b.reshape(-1) - c.matvec(sol.reshape(1, -1)).reshape(-1)
    return (r.norm() / b.norm()).item()


@pytest.mark.parametrize("make,restart", [
    (lambda: sphere_problem(0), 100), (lambda: sphere_problem(1), 3), (lambda: floating_shell_problem(2), 7),
    (lambda: coax_problem(0.012), 100), (lambda: coax_problem(0.012), 20), (lambda: coax_problem(0.0028), 100)])
def test_gmres_residual(bem, make, restart):
    p = make()
    print(f"[gpu-gmres] {p.name} N={p.n_tri} restart={restart}", flush=True)
    with bem.Context.from_problem(p, restart=restart) as c:
        c.assemble()
        for tol in (1e-10, 1e-4, 1e-10):
            sol, info = c.solve(p.body_V, tol=tol, max_iter=3000)
            assert info["converged"] and info["rel_residual"] <= tol
            assert _residual(c, p, sol) <= tol + 1e-13
            again, info2 = c.solve(p.body_V, tol=tol, max_iter=3000)
            assert info2["iters"] == info["iters"] and torch.equal(again, sol)


@pytest.mark.parametrize("limit", [1, 2, 5, 6, 7])
def test_gmres_iteration_limit(bem, limit):
    p = coax_problem(0.012)
    print(f"[gpu-gmres] limit {limit}", flush=True)
    with bem.Context.from_problem(p, restart=6) as c:
        c.assemble()
        sol, info = c.solve(p.body_V, tol=1e-10, max_iter=limit, raise_on_noconv=False)
        assert not info["converged"] and info["iters"] == limit
        assert abs(_residual(c, p, sol) - info["rel_residual"]) <= 1e-12
