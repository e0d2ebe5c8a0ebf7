"""The tridiagonal reduction of Rayleigh-Ritz at the edges of its forms: one, two or three
rows per lane (real n <= 64, 128, 192; complex n <= 64, 128), the panel form above, sizes off
the eight column groups, and blocks whose projected matrix has exactly zero columns (points
that no stencil line or projector couples), where a reflector is the identity.  Compared with
scipy's generalised eigenvalues of the oracle's projected pencil.  Both sides are backward
stable: the error of an eigenvalue is a small multiple of n eps |H| cond(X)^2, and a random
block of n <= 192 columns on 4896 points has cond(X)^2 < 3; the bar takes the factor 100."""
import numpy as np
import pytest
import scipy.linalg

torch = pytest.importorskip("torch")

from oracle.fd import apply_H
from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl
from tests.helpers import oracle_setup, to_dev, block_to_oracle

pytestmark = pytest.mark.gpu

EPS = np.finfo(np.float64).eps


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("points", [False, True])
@pytest.mark.parametrize("cplx,n", [(False, n) for n in (2, 7, 64, 65, 127, 128, 129, 191, 192, 193)] +
                         [(True, n) for n in (2, 9, 63, 64, 65, 128, 129)])
def test_rayleigh_ritz_at_the_edges(ctx, cplx, n, points):
    k = (0.1, 0.2, -0.1) if cplx else (0.0, 0.0, 0.0)
    cell, rng = wl.draw_cell(94, 70, (18, 16, 17), (9.0, 8.0, 8.5), 3, (0, 1), 2.5, 0)
    grid, V, P = oracle_setup(cell, k)
    if points:      # unit vectors, no two within a stencil's reach on one grid line
        X = np.zeros((n, cell.n_d))
        X[np.arange(n), (np.arange(n) * 18 + (np.arange(n) * 5) % 18)] = 1.0
    else:
        X = rng.standard_normal((n, cell.n_d))
        if cplx:
            X = X + 1j * rng.standard_normal((n, cell.n_d))
    if cplx:
        X = X.astype(np.complex128)
    h = sp.Hamiltonian(ctx, cell, sp.C128 if cplx else sp.R64, kpt=k)
    Xd = to_dev(X)
    ritz = torch.zeros(n, dtype=torch.float64, device="cuda")
    sp.rayleigh_ritz(h, Xd, ritz, sp.workspace(h, n, sp.OP_RR))
    B = X.T.copy()
    HB = apply_H(B, grid, V, P)
    A, G = B.conj().T @ HB, B.conj().T @ B
    want = scipy.linalg.eigvalsh((A + A.conj().T) / 2, (G + G.conj().T) / 2)
    width = np.abs(want).max() + np.linalg.norm(HB, axis=0).max() / np.linalg.norm(B, axis=0).min()
    tol = 100 * n * EPS * width * 3
    assert np.abs(ritz.cpu().numpy() - want).max() <= tol
    Q = block_to_oracle(Xd)
    assert np.abs(Q.conj().T @ Q - np.eye(n)).max() <= 100 * n * EPS * 3
    R = Q.conj().T @ apply_H(Q, grid, V, P)
    assert np.abs(R - np.diag(ritz.cpu().numpy())).max() <= tol
