"""Row form of the stencil step against the oracle: H X and the in-place recurrence at the
edges of its tiles (rows that no 16-byte chunk divides, tiles with rows past the grid,
lanes past the tile, the smallest grid it takes, rows wide enough for two halo chunks per
thread, FP32 and complex double rows that stay tiled), block pointers off 16-byte alignment,
leading dimensions above N_d, complex Bloch phases on every face, and several problems of different
sizes and chunk widths in one plan.
Tolerances: the ones of the tiled form (1e-12 of a column's norm in FP64 for H X, 1e-10
through a filter, 2e-5 / 2e-4 in FP32)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.fd import apply_H
from oracle.chefsi import cheb_filter
from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl
from tests.helpers import oracle_setup, colnorm_err, to_dev, block_to_oracle

pytestmark = pytest.mark.gpu

GRIDS = [((16, 16, 16), 24), ((24, 20, 18), 24), ((17, 19, 23), 20), ((45, 38, 17), 16), ((18, 50, 16), 16),
         ((96, 33, 16), 8), ((130, 18, 16), 6), ((20, 16, 40), 1), ((43, 48, 16), 160),
         ((58, 53, 17), 100)]
TYPES = {"r64": (sp.R64, torch.float64, 1e-12, 1e-10), "r32": (sp.R32, torch.float32, 2e-5, 2e-4),
         "c128": (sp.C128, torch.complex128, 1e-12, 1e-10), "c64": (sp.C64, torch.complex64, 2e-5, 2e-4)}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


def _problem(n, ns, cplx, seed):
    cell, rng = wl.draw_cell(95, seed, n, tuple(0.45 * v for v in n), 3, (0, 1), 2.0, ns)
    k = tuple(0.31 * (s + 1) * (-1) ** s / cell.L[s] for s in range(3)) if cplx else (0.0, 0.0, 0.0)
    X = rng.standard_normal((ns, cell.n_d))
    if cplx:
        X = X + 1j * rng.standard_normal((ns, cell.n_d))
    return cell, k, X


def _padded(X, tdt, pad, shift):
    """Device block with leading dimension N_d + pad, starting `shift` elements into an
    allocation."""
    ns, nd = X.shape
    buf = torch.full((ns * (nd + pad) + shift,), 7.0, dtype=tdt, device="cuda:0")
    t = buf[shift:].view(ns, nd + pad)
    t[:, :nd] = to_dev(X).to(tdt)
    return t


@pytest.mark.parametrize("pad,shift", [(0, 0), (5, 1)])
@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("n,ns", GRIDS)
def test_row_form(ctx, n, ns, dt, pad, shift):
    code, tdt, tol_h, tol_f = TYPES[dt]
    cell, k, X = _problem(n, ns, dt.startswith("c"), sum(n))
    grid, V, P = oracle_setup(cell, k)
    ham = sp.Hamiltonian(ctx, cell, code, kpt=k)
    Xd = _padded(X, tdt, pad, shift)
    Yd = _padded(np.zeros_like(X), tdt, pad, shift)
    Xr = block_to_oracle(Xd)[:grid.n_d]
    sp.fd_hamiltonian_apply(ham, Xd, Yd, sp.workspace(ham, ns, sp.OP_APPLY))
    Y = block_to_oracle(Yd)
    assert colnorm_err(Y[:grid.n_d], apply_H(Xr, grid, V, P)) < tol_h
    np.testing.assert_array_equal(Y[grid.n_d:], 7.0)   # nothing past the block's rows
    lmax = 1.5 * np.pi ** 2 * sum((cell.n[s] / cell.L[s]) ** 2 for s in range(3)) / 2
    for degree in (4, 5):
        F = Xd.clone()
        sp.chebyshev_filter(ham, F, degree, 0.2 * lmax, lmax, sp.workspace(ham, ns, sp.OP_FILTER))
        ref = cheb_filter(Xr, grid, V, P, degree, 0.2 * lmax, lmax)
        assert colnorm_err(block_to_oracle(F)[:grid.n_d], ref) < tol_f


@pytest.mark.parametrize("dt", ["r64", "c128", "r32"])
def test_row_form_uneven_plan(ctx, dt):
    code, tdt, _, tol_f = TYPES[dt]
    probs, hams, Xs, deg = [], [], [], []
    for i, (n, ns, d) in enumerate([((40, 36, 32), 12, 6), ((17, 16, 18), 20, 5), ((24, 24, 24), 9, 3)]):
        cell, k, X = _problem(n, ns, dt.startswith("c"), 7 + i)
        probs.append((oracle_setup(cell, k), X))
        hams.append(sp.Hamiltonian(ctx, cell, code, kpt=k))
        Xs.append(to_dev(X).to(tdt))
        deg.append(d)
    plan = sp.FilterPlan(ctx, hams, Xs, deg)
    for _ in range(2):   # the captured graph, replayed on new data
        for x, (_, X) in zip(Xs, probs):
            x.copy_(to_dev(X))
        plan.run([10.0, 12.0, 9.0], [60.0, 70.0, 65.0])
        for i, ((grid, V, P), X) in enumerate(probs):
            ref = cheb_filter(X.T.astype(block_to_oracle(Xs[i]).dtype), grid, V, P, deg[i], [10.0, 12.0, 9.0][i],
                              [60.0, 70.0, 65.0][i])
            assert colnorm_err(block_to_oracle(Xs[i]), ref) < tol_f
    plan.close()
