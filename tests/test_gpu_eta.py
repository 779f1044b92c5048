"""Far from the usual eta = 6 of the Sec. 4 classification, against the oracle with the same eta.

At 40 nearly every pair takes its closed form, so that a point's list of near pairs fills a wave's LDS
list several times over."""

import numpy as np
import pytest

from workloads import electrode_line_starts, sphere_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_12663_amd as bem
    return bem


@pytest.mark.parametrize("eta", [40.0])
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
