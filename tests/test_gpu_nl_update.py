"""The filter's one-pass projector update (scatter of a step with the gather of the next)
against the oracle where it is taken (2 x 256 pairs of atoms and four orbitals): supports that
share most of their nodes and supports that share few, one and four projectors per atom, a
ragged last block of orbitals, padded and off-aligned blocks, degrees 1, 2 and 5 (no update,
one, several), and a plan whose problems end at different steps.
Tolerances: those of the filter elsewhere, 1e-10 of a column's norm in FP64, 2e-4 in FP32."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.chefsi import cheb_filter
from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl
from tests.helpers import oracle_setup, colnorm_err, to_dev, block_to_oracle

pytestmark = pytest.mark.gpu

TYPES = {"r64": (sp.R64, torch.float64, 1e-10), "r32": (sp.R32, torch.float32, 2e-4),
         "c128": (sp.C128, torch.complex128, 1e-10), "c64": (sp.C64, torch.complex64, 2e-4)}
# grid, spacing, atoms, states: crowded, sparse, nearly every node in many supports
CELLS = [((18, 17, 16), 0.45, 22, 93), ((28, 26, 24), 0.5, 8, 253), ((16, 18, 16), 0.3, 40, 49)]


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


def _problem(n, h, atoms, ns, ls, cplx, seed):
    cell, rng = wl.draw_cell(96, seed, n, tuple(h * v for v in n), atoms, ls, 2.0, ns)
    k = tuple(0.31 * (s + 1) * (-1) ** s / cell.L[s] for s in range(3)) if cplx else (0.0, 0.0, 0.0)
    X = rng.standard_normal((ns, cell.n_d))
    if cplx:
        X = X + 1j * rng.standard_normal((ns, cell.n_d))
    lmax = 1.5 * np.pi ** 2 / h ** 2
    return cell, k, X, 0.2 * lmax, lmax


@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("ls", [(0,), (0, 1)])
@pytest.mark.parametrize("n,h,atoms,ns", CELLS)
def test_update_in_the_filter(ctx, n, h, atoms, ns, ls, dt):
    code, tdt, tol = TYPES[dt]
    cell, k, X, lcut, lmax = _problem(n, h, atoms, ns, ls, dt.startswith("c"), sum(n) + len(ls))
    grid, V, P = oracle_setup(cell, k)
    ham = sp.Hamiltonian(ctx, cell, code, kpt=k)
    work = sp.workspace(ham, ns, sp.OP_FILTER)
    for degree in (1, 2, 5):
        buf = torch.full((ns * (cell.n_d + 3) + 1,), 7.0, dtype=tdt, device="cuda:0")
        F = buf[1:].view(ns, cell.n_d + 3)
        F[:, :cell.n_d] = to_dev(X).to(tdt)
        ref = cheb_filter(block_to_oracle(F)[:cell.n_d], grid, V, P, degree, lcut, lmax)
        sp.chebyshev_filter(ham, F, degree, lcut, lmax, work)
        out = block_to_oracle(F)
        assert colnorm_err(out[:cell.n_d], ref) < tol
        np.testing.assert_array_equal(out[cell.n_d:], 7.0)


@pytest.mark.parametrize("use_graph", [False, True])
@pytest.mark.parametrize("dt", ["r64", "c128", "r32"])
def test_update_in_a_plan(ctx, dt, use_graph):
    code, tdt, tol = TYPES[dt]
    probs = [_problem(n, h, atoms, ns, ls, dt.startswith("c"), 7 + i) for i, (n, h, atoms, ns, ls) in enumerate(
        [((18, 17, 16), 0.45, 22, 70, (0,)), ((20, 16, 22), 0.5, 5, 61, (0, 1)), ((16, 18, 16), 0.3, 9, 24, (0, 1))])]
    degs = [6, 3, 1]
    hams = [sp.Hamiltonian(ctx, c, code, kpt=k) for c, k, *_ in probs]
    Xs = [to_dev(X).to(tdt) for _, _, X, _, _ in probs]
    refs = []
    for (c, k, _, lcut, lmax), X, d in zip(probs, Xs, degs):
        grid, V, P = oracle_setup(c, k)
        refs.append(cheb_filter(block_to_oracle(X), grid, V, P, d, lcut, lmax))
    start = [X.clone() for X in Xs]
    plan = sp.FilterPlan(ctx, hams, Xs, degs, use_graph=use_graph)
    for _ in range(3):
        for X, s in zip(Xs, start):
            X.copy_(s)
        plan.run([p[3] for p in probs], [p[4] for p in probs])
        for X, ref in zip(Xs, refs):
            assert colnorm_err(block_to_oracle(X), ref) < tol
