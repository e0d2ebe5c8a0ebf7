"""A context that autotunes gives the results of one that does not, bit by bit: a node's arithmetic
is the same in every row plan, in every tile shape, and the tuner stays within the form that the
step takes.  Row form (16-byte, narrower and one-value chunks, all types), tiled form by stencil
order and by Dirichlet faces, and plans of one and of several chunk widths, with and without a
captured graph."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl
from tests.helpers import to_dev

pytestmark = pytest.mark.gpu

TYPES = {"r64": sp.R64, "r32": sp.R32, "c128": sp.C128, "c64": sp.C64}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


def _problem(ctx, n, ns, dt, n_o=6, bc=(0, 0, 0)):
    cplx = dt.startswith("c")
    cell, rng = wl.draw_cell(91, sum(n) + ns, n, tuple(0.5 * v for v in n), 3, (0, 1), 2.0, ns)
    cell.bc = bc
    k = (0.1, -0.2, 0.15) if cplx else (0.0, 0.0, 0.0)
    X = rng.standard_normal((ns, cell.n_d)) + (1j * rng.standard_normal((ns, cell.n_d)) if cplx else 0.0)
    return sp.Hamiltonian(ctx, cell, TYPES[dt], kpt=k, n_o=n_o), to_dev(X).to(sp.TORCH_DTYPE[TYPES[dt]])


def _tuned(ctx, run):
    want = run()
    sp.set_autotune(ctx, True)
    try:
        first, later = run(), run()
    finally:
        sp.set_autotune(ctx, False)
    torch.cuda.synchronize()
    for a in (first, later):
        assert all(torch.equal(u, v) for u, v in zip(want, a))


@pytest.mark.parametrize("n,ns,dt,n_o,bc", [
    ((48, 44, 40), 40, "r64", 6, (0, 0, 0)), ((45, 38, 51), 30, "r64", 6, (0, 0, 0)), ((40, 40, 40), 56, "r32", 6, (0, 0, 0)),
    ((43, 33, 30), 50, "r32", 6, (0, 0, 0)), ((32, 30, 36), 24, "c128", 6, (0, 0, 0)), ((45, 38, 33), 20, "c64", 6, (0, 0, 0)),
    ((64, 40, 30), 32, "r64", 4, (0, 0, 0)), ((40, 33, 36), 48, "r64", 6, (0, 1, 1)), ((40, 33, 36), 48, "c64", 5, (0, 0, 1))])
def test_single_calls(ctx, n, ns, dt, n_o, bc):
    if dt.startswith("c") and any(bc):
        cell_k = (0.1, -0.2, 0.0)   # no phase across a Dirichlet face
        cell, rng = wl.draw_cell(91, 5, n, tuple(0.5 * v for v in n), 3, (0, 1), 2.0, ns)
        cell.bc = bc
        ham = sp.Hamiltonian(ctx, cell, TYPES[dt], kpt=cell_k, n_o=n_o)
        X = to_dev(rng.standard_normal((ns, cell.n_d)) + 1j * rng.standard_normal((ns, cell.n_d))).to(torch.complex64)
    else:
        ham, X = _problem(ctx, n, ns, dt, n_o, bc)

    def run():
        Y, F = torch.zeros_like(X), X.clone()
        sp.fd_hamiltonian_apply(ham, X, Y, sp.workspace(ham, ns, sp.OP_APPLY))
        sp.chebyshev_filter(ham, F, 5, 10.0, 60.0, sp.workspace(ham, ns, sp.OP_FILTER))
        return Y, F

    _tuned(ctx, run)


@pytest.mark.parametrize("graph", [False, True])
@pytest.mark.parametrize("dt,spec", [("r64", [((40, 36, 32), 30), ((17, 16, 18), 20), ((24, 24, 24), 9)]),
                                     ("c128", [((32, 32, 32), 40), ((32, 32, 32), 40)]),
                                     ("r32", [((40, 33, 36), 24), ((42, 20, 20), 12), ((43, 18, 16), 12)]),
                                     ("r64", [((40, 36, 32), 30), ((12, 14, 10), 20)])])
def test_plans(ctx, dt, spec, graph):
    probs = [_problem(ctx, n, ns, dt) for n, ns in spec]
    deg = [5, 4, 3][:len(probs)]

    def run():
        Xs = [X.clone() for _, X in probs]
        plan = sp.FilterPlan(ctx, [h for h, _ in probs], Xs, deg, use_graph=graph)
        plan.run([10.0] * len(probs), [60.0] * len(probs))
        torch.cuda.synchronize()
        plan.close()
        return Xs

    _tuned(ctx, run)
