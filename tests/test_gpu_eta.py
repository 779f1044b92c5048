"""Far from the usual eta = 6 of the Sec. 4 classification, against the oracle with the same eta.

At 40 nearly every pair takes its closed form, so that a point's list of near pairs fills a wave's LDS
list several times over.  At 1 and 1.5 regular pairs come as close as a circumradius or two, where the
rule about the centroid takes its node distances from larger numbers than they are."""

import numpy as np
import pytest

from workloads import coax_problem, electrode_line_starts, floating_shell_problem, sphere_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_12663_amd as bem
    return bem


@pytest.mark.parametrize("make", [lambda: floating_shell_problem(2), lambda: coax_problem(0.018)])
@pytest.mark.parametrize("eta", [1.0, 1.5])
def test_rows_and_field(bem, oracle_mod, make, eta):
    """Every row to 1e-12 of its largest entry; potential and field at and off the panels to 1e-10."""
    p = make()
    print(f"[gpu-eta] rows N={p.n_tri} eta={eta}", flush=True)
    o = oracle_mod.Oracle(p, eta=eta)
    cen = p.vert[p.tri].mean(axis=1)
    x = np.concatenate([1.0 + 0.3 * np.sin(cen @ [1.0, 2.0, 3.0]), np.zeros(p.n_float)])
    with bem.Context.from_problem(p, eta=eta) as c:
        c.assemble()
        A, G = o.assemble(), c.copy_rows(0, c.n).cpu().numpy()
        assert (np.abs(G - A) <= 1e-12 * np.abs(A).max(axis=1, keepdims=True)).all()
        for pts, on in ((cen, np.arange(p.n_tri, dtype=np.int32)), (cen * 1.003, None), (cen * 1.1, None)):
            phi, E = c.eval_field(torch.tensor(x, device="cuda"), pts, on_panel=on)
            for got, want in zip((phi[0], E[0]), o.eval(x, pts, on_panel=on)):
                assert np.abs(got.cpu().numpy() - want).max() <= 1e-10 * np.abs(want).max()


@pytest.mark.parametrize("eta", [1.0, 1.5])
def test_nodal_rows(bem, oracle_mod, eta):
    p = floating_shell_problem(2)
    print(f"[gpu-eta] nodal rows N={p.n_tri} eta={eta}", flush=True)
    with bem.Context.from_problem(p, eta=eta, basis=bem.BASIS_LINEAR, constraint_form=1) as c:
        c.assemble()
        A, G = oracle_mod.Oracle(p, eta=eta, constraint_form=1).p1_assemble(), c.copy_rows(0, c.n).cpu().numpy()
    assert (np.abs(G - A) <= 1e-12 * np.abs(A).max(axis=1, keepdims=True)).all()


@pytest.mark.parametrize("eta", [1.5, 40.0])
def test_gradient(bem, oracle_mod, eta):
    """dJ along a direction of the vertices and potentials, 1e-8 of the norms' product (the bar of the
    gradient tests), from the oracle's dual numbers."""
    p = sphere_problem(2, V0=50.0)
    print(f"[gpu-eta] gradient N={p.n_tri} eta={eta}", flush=True)
    L, kw = 4, dict(h=1e-3, max_steps=12, e_min=1e-3)
    starts, panel, bary = electrode_line_starts(p, L, seed=6)
    g = np.random.default_rng(11).uniform(0.5, 1.5, L)
    with bem.Context.from_problem(p, eta=eta) as c:
        c.assemble()
        sol, _ = c.solve(p.body_V, tol=1e-13, max_iter=20000)
        tp = bem.trace_params(**kw)
        I, ns, _, _ = c.streamer_integral(sol, starts, tp)
        dvert, dV = (t.cpu().numpy() for t in c.streamer_grad(sol, starts, g, tp, start_panel=panel, start_bary=bary)[:2])
    rng = np.random.default_rng(8)
    dv, dW = rng.standard_normal(p.vert.shape), rng.standard_normal(p.n_body)
    o = oracle_mod.Oracle(p, eta=eta)
    Io, dI, _, _, rc = o.dual_streamer(dv, p.body_V, dW, panel, bary, oracle_mod.trace_params(**kw), ns.cpu().numpy())
    assert rc == 0
    assert np.abs(I.cpu().numpy() - Io).max() <= 1e-10 * np.abs(Io).max()
    got = np.sum(dvert * dv) + np.sum(dV.reshape(-1) * dW)
    scale = np.linalg.norm(dvert) * np.linalg.norm(dv) + np.linalg.norm(dV) * np.linalg.norm(dW)
    assert abs(got - np.dot(g, dI)) <= 1e-8 * scale
