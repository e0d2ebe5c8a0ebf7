"""Rayleigh-Ritz of badly scaled blocks at the sizes where the Cholesky block (16 x 16 sub-blocks,
64 x 64 blocks) and the condition estimate (eight lanes a row up to 128 states, LDS up to about
100 real) change form: orthonormality and the projected matrix against the block's own H X.
Columns are scaled over eight orders of magnitude, which the column-scaled factorisation removes;
the block is random, so cond(X)^2 < 3 after scaling and the bars are 100 n eps of it, as for the
tridiagonal reduction.  A block with two equal columns takes the shifted path and must still
return an orthonormal basis."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("cplx,n", [(False, n) for n in (1, 3, 15, 16, 17, 48, 63, 64, 65, 99, 128, 129)] +
                         [(True, n) for n in (1, 16, 33, 64, 65, 81, 128, 129)])
def test_scaled_columns(ctx, cplx, n):
    cell, rng = wl.draw_cell(94, 71, (18, 16, 17), (9.0, 8.0, 8.5), 3, (0, 1), 2.5, 0)
    k = (0.1, 0.2, -0.1) if cplx else (0.0, 0.0, 0.0)
    X = rng.standard_normal((n, cell.n_d)) + (1j * rng.standard_normal((n, cell.n_d)) if cplx else 0.0)
    X = torch.from_numpy(X * 10.0 ** rng.uniform(-4, 4, (n, 1))).cuda()
    ham = sp.Hamiltonian(ctx, cell, sp.C128 if cplx else sp.R64, kpt=k)
    ritz = torch.zeros(n, dtype=torch.float64, device="cuda")
    sp.rayleigh_ritz(ham, X, ritz, sp.workspace(ham, n, sp.OP_RR))
    HX = torch.empty_like(X)
    sp.fd_hamiltonian_apply(ham, X, HX, sp.workspace(ham, n, sp.OP_APPLY))
    Q, HQ = X.cpu().numpy(), HX.cpu().numpy()
    width = np.linalg.norm(HQ, axis=1).max()
    assert np.abs(Q.conj() @ Q.T - np.eye(n)).max() <= 300 * n * EPS
    assert np.abs(Q.conj() @ HQ.T - np.diag(ritz.cpu().numpy())).max() <= 300 * n * EPS * width


@pytest.mark.parametrize("n", [40, 100])
def test_dependent_columns(ctx, n):
    cell, rng = wl.draw_cell(94, 71, (18, 16, 17), (9.0, 8.0, 8.5), 3, (0, 1), 2.5, 0)
    X = rng.standard_normal((n, cell.n_d))
    X[n // 2] = X[3] * (1.0 + 1e-9 * rng.standard_normal(cell.n_d))
    X = torch.from_numpy(X).cuda()
    ham = sp.Hamiltonian(ctx, cell, sp.R64)
    ritz = torch.zeros(n, dtype=torch.float64, device="cuda")
    sp.rayleigh_ritz(ham, X, ritz, sp.workspace(ham, n, sp.OP_RR))
    Q = X.cpu().numpy()
    assert np.abs(Q @ Q.T - np.eye(n)).max() <= 300 * n * EPS
