"""Field evaluation at the edges of its split (one point per lane over ranges of panels, then one
wave per point for the near pairs) against the FP64 oracle.

Point counts around a wave, a block and a wave's four points; panel ranges of one word of marks, of
all panels and ones that do not divide the panel count; points on panels (with and without
`on_panel`), close to them and far off, so that a point has no near pair, a few, or more than one
round of a wave.  Relative 1e-10 (the workload's FP64 bar) on potential and field."""

import numpy as np
import pytest

import oracle
from workloads import coax_problem, sphere_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_12663_amd as bem
    return bem


@pytest.mark.parametrize("make,P,blocks", [
    (lambda: sphere_problem(0), 1, 64), (lambda: sphere_problem(1), 65, 65536), (lambda: sphere_problem(3), 255, 64),
    (lambda: sphere_problem(3), 257, 65536), (lambda: coax_problem(0.012), 4, 2048), (lambda: coax_problem(0.012), 513, 300)])
@pytest.mark.parametrize("eta", [6.0, 60.0])
def test_field_at_split_edges(bem, make, P, blocks, eta):
    p = make()
    print(f"[gpu-eval] {p.name} N={p.n_tri} P={P} blocks={blocks} eta={eta}", flush=True)
    rng = np.random.default_rng(P)
    cen = p.vert[p.tri].mean(axis=1)
    size = np.abs(p.vert).max()
    x = np.concatenate([1.0 + 0.3 * np.sin(cen @ rng.uniform(-1.0, 1.0, 3) / size), np.zeros(p.n_float)])
    on = rng.integers(0, p.n_tri, P).astype(np.int32)
    pts = cen[on].copy()
    on[rng.random(P) < 0.5] = -1
    move = on < 0
    pts[move] += size * rng.choice([1e-3, 0.1, 30.0], (P, 1))[move] * rng.standard_normal((P, 3))[move]
    o = oracle.Oracle(p, eta=eta)
    with bem.Context.from_problem(p, eta=eta) as c:
        c.set_tuning("eval_blocks", blocks)
        for op in (on, None):
            q = pts if op is not None else pts[move]
            if len(q) == 0:
                continue
            po, Eo = o.eval(x, q, on_panel=op)
            phi, E = c.eval_field(torch.tensor(x, device="cuda"), q, on_panel=op)
            none, E2 = c.eval_field(torch.tensor(x, device="cuda"), q, on_panel=op, want_phi=False)
            assert none is None
            for got, want in ((phi[0], po), (E[0], Eo), (E2[0], Eo)):
                d = np.abs(got.cpu().numpy() - want)
                assert d.max() <= 1e-10 * np.abs(want).max()


def test_refused_points(bem):
    """A non-finite coordinate or a panel out of range anywhere in the list is refused before anything runs."""
    p = sphere_problem(2)
    print("[gpu-eval] refused points", flush=True)
    cen = np.tile(p.vert[p.tri].mean(axis=1), (2, 1))
    on = np.tile(np.arange(p.n_tri, dtype=np.int32), 2)
    with bem.Context.from_problem(p) as c:
        sol = torch.ones(p.n_tri, dtype=torch.float64, device="cuda")
        c.eval_field(sol, cen, on_panel=on)
        for row, value in ((0, np.nan), (len(cen) - 1, np.inf), (300, -np.inf)):
            bad = cen.copy()
            bad[row, row % 3] = value
            with pytest.raises(bem.BemError, match="non-finite point coordinate"):
                c.eval_field(sol, bad, on_panel=on)
        for row, value in ((0, -2), (len(on) - 1, p.n_tri), (300, 2**31 - 1)):
            bad = on.copy()
            bad[row] = value
            with pytest.raises(bem.BemError, match="on_panel entry out of range"):
                c.eval_field(sol, cen, on_panel=bad)
        c.eval_field(sol, cen, on_panel=on)
