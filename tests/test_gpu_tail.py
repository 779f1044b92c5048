"""trace_mode 0 on both sides of the cluster layout.

Without it (trace_cluster 0, as on a device that refuses the cooperative launch) the lines run in the
two-kernel layout and then its one-launch tail: the handover between the two, in FP64 and with the nodal
basis, with counters that show that both parts ran.  With it (the default): the stops at a line's first
stage, lines of several load cases, and many lines with many near panels, which go to the two-kernel
layout.  Step counts and stop codes exact, integrals 1e-10 relative (the
workload's FP64 bar), against the oracle."""

import numpy as np
import pytest

import oracle
from workloads import coax_conductors_problem, coax_problem, electrode_line_starts, sphere_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def bem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_12663_amd as bem
    return bem


@pytest.fixture(scope="module")
def coax():
    """(problem, oracle, density) of the 2,192-panel coax."""
    p = coax_problem(0.012)
    o = oracle.Oracle(p)
    return p, o, np.linalg.solve(o.assemble(), o.rhs(p.body_V))


def _compare(got, want):
    I, ns, st = (t.cpu().numpy() for t in got[:3])
    nso, sto, Io = want[:3]
    assert np.array_equal(ns, nso) and np.array_equal(st, sto)
    assert np.abs(I - Io).max() <= 1e-10 * np.abs(Io).max()
    return ns, st


@pytest.mark.parametrize("loop", [0, 64])
def test_handover_on_a_hit_step(bem, coax, loop):
    """The tail's first launch evaluates the end point of step 8 (pass 32), where most of the 32 lines have
    crossed the shell: it has to test that step's segment."""
    p, o, x = coax
    print(f"[gpu-tail] hit step, trace_loop {loop}", flush=True)
    starts, _, _ = electrode_line_starts(p, 32, seed=3)
    kw = dict(h=0.0105, max_steps=12)
    with bem.Context.from_problem(p) as c:
        for k, v in dict(trace_cluster=0, trace_tail=4096, trace_loop=loop).items():
            c.set_tuning(k, v)
        got = c.streamer_integral(torch.tensor(x, device="cuda"), starts, bem.trace_params(**kw))
        assert c.counter("trace_far_launches") > 0 and c.counter("trace_pass_launches") > 0
    ns, st = _compare(got, o.trace(x, starts, oracle.trace_params(**kw)))
    assert ((ns == 7) & (st == 1)).sum() >= 20


@pytest.mark.parametrize("tuning", [dict(trace_tail=8), dict(trace_tail=16), dict(trace_tail=16, trace_loop=0)],
                         ids=["tail8", "tail16", "tail16_stage"])
def test_handover_to_the_tail(bem, coax, tuning):
    """16 lines that end on the shell or the ring or run out of steps, handed over at 8 or 16 live lines."""
    p, o, x = coax
    print(f"[gpu-tail] {tuning}", flush=True)
    starts, _, _ = electrode_line_starts(p, 16, seed=21)
    kw = dict(h=1e-3, max_steps=200)
    with bem.Context.from_problem(p) as c:
        for k, v in dict(trace_cluster=0, **tuning).items():
            c.set_tuning(k, v)
        got = c.streamer_integral(torch.tensor(x, device="cuda"), starts, bem.trace_params(**kw))
        assert c.counter("trace_far_launches") > 0 and c.counter("trace_pass_launches") > 0
    ns, st = _compare(got, o.trace(x, starts, oracle.trace_params(**kw)))
    assert len(set(st.tolist())) >= 2


def test_handover_nodal(bem):
    p = coax_conductors_problem(0.012)
    print(f"[gpu-tail] nodal N={p.n_tri}", flush=True)
    u = np.concatenate([60.0 + 0.0 * p.vert[:, 0] + 200.0 * p.vert[:, 2], np.zeros(p.n_float)])
    starts, _, _ = electrode_line_starts(p, 16, seed=5)
    kw = dict(h=1e-3, max_steps=40)
    with bem.Context.from_problem(p, basis=bem.BASIS_LINEAR, constraint_form=1) as c:
        c.set_tuning("trace_cluster", 0)
        got = c.streamer_integral(torch.tensor(u[None], device="cuda"), starts, bem.trace_params(**kw))
        assert c.counter("trace_far_launches") > 0 and c.counter("trace_pass_launches") > 0
    _compare(got, oracle.Oracle(p, constraint_form=1).p1_trace(u, starts, oracle.trace_params(**kw)))


def _default(bem, c, *args, **kw):
    """A run of the default layout, which is the cluster layout: one launch and no passes."""
    c.reset_stats()
    got = c.streamer_integral(*args, **kw)
    assert c.counter("trace_pass_launches") == 1 and c.counter("trace_far_launches") == 0
    return got


@pytest.mark.parametrize("nodal", [False, True])
def test_stops_of_the_default(bem, nodal):
    """One step; inward lines that hit the electrode before a step; a field below e_min everywhere; a density
    that is not finite; no line at all."""
    p = sphere_problem(2, V0=50.0)
    print(f"[gpu-tail] stops nodal={nodal}", flush=True)
    kw = dict(basis=bem.BASIS_LINEAR, constraint_form=1) if nodal else {}
    with bem.Context.from_problem(p, **kw) as c:
        sol = torch.full((1, c.n), 60.0, dtype=torch.float64, device="cuda")
        starts, _, _ = electrode_line_starts(p, 70, seed=1)
        tp = dict(h=1e-3, max_steps=5)
        for extra, steps, code in ((dict(max_steps=1), 1, 0), (dict(direction=-1), 0, 1), (dict(e_min=1e6), 0, 4)):
            I, ns, st, _ = _default(bem, c, sol, starts, bem.trace_params(**{**tp, **extra}))
            assert (ns == steps).all() and (st == code).all()
        bad = sol.clone()
        bad[0, 7] = float("nan")
        I, ns, st, _ = _default(bem, c, bad, starts, bem.trace_params(**tp))
        assert (ns == 0).all() and (st == 5).all()
        assert c.streamer_integral(sol, np.zeros((0, 3)), bem.trace_params(**tp))[1].numel() == 0


def test_load_cases_of_the_default(bem, coax):
    """Lines that belong to three load cases in turn."""
    p, o, x = coax
    print("[gpu-tail] load cases", flush=True)
    xs = np.outer([0.7, 1.0, 1.6], x)
    starts, _, _ = electrode_line_starts(p, 9, seed=11)
    owner = np.array([0, 1, 2] * 3, dtype=np.int32)
    kw = dict(h=1e-3, max_steps=60)
    with bem.Context.from_problem(p) as c:
        got = _default(bem, c, torch.tensor(xs, device="cuda"), starts, bem.trace_params(**kw), line_rhs=owner)
    for r in range(3):
        sel = np.nonzero(owner == r)[0]
        _compare([t[torch.tensor(sel, device="cuda")] for t in got[:3]],
                 o.trace(xs[r], starts[sel], oracle.trace_params(**kw)))


@pytest.mark.parametrize("nodal,L", [(False, 4096), (True, 1100)])
def test_many_lines_with_many_near_panels(bem, nodal, L):
    """At eta = 40 every panel of this sphere is near.  That many lines take the two-kernel layout (the cluster
    layout is slower), unless trace_blocks asks for the other; few of them, and as many at the usual eta,
    take the cluster layout.  The same results either way."""
    p = sphere_problem(2, V0=50.0)
    print(f"[gpu-tail] many lines nodal={nodal} L={L}", flush=True)
    x = np.concatenate([60.0 * (1.0 + 0.3 * np.sin((p.vert if nodal else p.vert[p.tri].mean(axis=1)) @ [1.0, 2.0, 0.5])),
                        np.zeros(p.n_float)])
    starts, _, _ = electrode_line_starts(p, L, seed=13)
    kw = dict(h=1e-3, max_steps=2)
    base = dict(basis=bem.BASIS_LINEAR, constraint_form=1) if nodal else {}
    sol, tp = torch.tensor(x[None], device="cuda"), bem.trace_params(**kw)
    for eta, few, blocks, cluster in ((40.0, L, 0, False), (40.0, L, 8, True), (40.0, 200, 0, True), (6.0, L, 0, True)):
        o = oracle.Oracle(p, eta=eta, constraint_form=1)
        with bem.Context.from_problem(p, eta=eta, **base) as c:
            c.set_tuning("trace_blocks", blocks)
            got = c.streamer_integral(sol, starts[:few], tp)
            assert (c.counter("trace_far_launches") == 0) == cluster
        _compare(got, (o.p1_trace if nodal else o.trace)(x, starts[:few], oracle.trace_params(**kw)))
