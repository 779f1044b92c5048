"""Mixed precision with several load cases: the results keep their bits.

The inner products of the batched solve take FP32 inputs, so the order of the FP64 sums around them
decides the last digits that the tolerance leaves open (1e-9 to 1e-8 of the solution); a change of that
order, or of one ulp in the operator, shows in these checksums and nowhere in a residual.  SHA-256 of the
solutions' bytes, taken with the library as of commit b7fca98, whose sums run one after another over the
split of each dot product; meshes with and without floating bodies.  Vertices are on a
grid of 2^-24 and line starts on one of 2^-40, so that the inputs are the same on every host."""

import hashlib

import numpy as np
import pytest

from workloads import coax_conductors_problem, coax_problem, electrode_line_starts, floating_shell_problem, sphere_problem

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

MESHES = {
    "sphere3": lambda: sphere_problem(3, V0=50.0),                # 1,280 panels, no floating body
    "shell2": lambda: floating_shell_problem(2, V0=80.0),         # 960 panels, one floating body
    "coax": lambda: coax_problem(0.012),                          # 2,192 panels, floating ring and interface
    "conductors": lambda: coax_conductors_problem(0.008),         # nodal basis: 1,912 vertices, net-charge row
}


def on_grid(p):
    p.vert = np.round(p.vert * 2.0 ** 24) / 2.0 ** 24
    return p


def potentials(p, nrhs):
    V = np.tile(p.body_V, (nrhs, 1)).astype(np.float64)
    return V * np.random.default_rng(nrhs).uniform(0.8, 1.6, (nrhs, 1))


def checksum(t):
    return hashlib.sha256(np.ascontiguousarray(t.cpu().numpy()).tobytes()).hexdigest()[:16]


def solve(bem, mesh, nrhs, lines=0, **kw):
    p = on_grid(MESHES[mesh]())
    with bem.Context.from_problem(p, precision=bem.MIXED, **kw) as c:
        c.assemble()
        sol, info = c.solve(potentials(p, nrhs), tol=1e-8)
        if lines == 0:
            return checksum(sol), info["iters"]
        starts = np.round(electrode_line_starts(p, lines, seed=nrhs)[0] * 2.0 ** 40) / 2.0 ** 40
        owner = torch.tensor((np.arange(lines) % nrhs).astype(np.int32), device="cuda")
        h = 1e-4 if mesh == "coax" else 1e-3
        total = c.streamer_integral(sol, starts, bem.trace_params(h=h, max_steps=60), line_rhs=owner)[0]
        return checksum(sol), checksum(total)


@pytest.fixture(scope="module")
def bem():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2003_12663_amd as bem
    return bem


# (checksum of the solutions, iterations)
SOLUTIONS = {
    ("sphere3", 2): ("392c025baf6e8c18", 18), ("sphere3", 5): ("106c85d7b39465c5", 18),
    ("sphere3", 64): ("6ba1c2342b05621a", 18), ("shell2", 2): ("17cb26209bd9206f", 22),
    ("shell2", 5): ("f0270857440e6dd5", 22), ("shell2", 64): ("ad248ea05c7e2964", 22),
    ("coax", 2): ("64a97b0b92360273", 44), ("coax", 5): ("375be4d7dcd14b88", 44),
    ("coax", 64): ("cd97fa6cb65359a8", 44),
}
# (checksum of the solutions, of the integrals)
LINES = {
    ("sphere3", 5): ("106c85d7b39465c5", "0b9cbc9e4fe5b9cd"),
    ("coax", 5): ("375be4d7dcd14b88", "9baf1ada9719a565"),
}


@pytest.mark.parametrize("mesh,nrhs", sorted(SOLUTIONS))
def test_solutions(bem, mesh, nrhs):
    print(f"[gpu-mixed-cases] {mesh} rhs={nrhs}", flush=True)
    assert solve(bem, mesh, nrhs) == SOLUTIONS[mesh, nrhs]


@pytest.mark.parametrize("mesh,nrhs", sorted(LINES))
def test_lines(bem, mesh, nrhs):
    """The integrals of 30 lines followed with those solutions."""
    print(f"[gpu-mixed-cases] lines {mesh} rhs={nrhs}", flush=True)
    assert solve(bem, mesh, nrhs, lines=30) == LINES[mesh, nrhs]


NODAL = {
    ("conductors", 2): ("f30685ac7a1ea230", 44), ("conductors", 5): ("b189a552328b308a", 44),
    ("conductors", 64): ("15a430ce238210b4", 44), ("shell2", 2): ("221fc9c8e20933b7", 19),
    ("shell2", 5): ("0b25a22be3dd3ab2", 19), ("shell2", 64): ("27cf965e50a2354d", 19),
}


@pytest.mark.parametrize("mesh,nrhs", sorted(NODAL))
def test_nodal_solutions(bem, mesh, nrhs):
    """The nodal basis: vertex rows in FP32 from FP64 sums over the rule's nodes, and a constraint row with
    (shell2) and without a K' term."""
    print(f"[gpu-mixed-cases] nodal {mesh} rhs={nrhs}", flush=True)
    assert solve(bem, mesh, nrhs, basis=bem.BASIS_LINEAR, constraint_form=int(mesh != "shell2")) == NODAL[mesh, nrhs]
