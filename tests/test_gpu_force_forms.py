"""Atomic forces at the edges of their kernels' forms: the non-local force with unrolled 12th-order
taps on grids as small as the taps allow, with every face crossed, against the same grid's
general form through a 10th-order stencil, each against the oracle; blocks of which some
orbitals are unoccupied and hold NaN; the local force of wells that are wider and narrower than
the cell, so that boxes wrap several times or hold a plane per work-group.
Bars: those of the other force tests, 1e-11 (non-local) and 1e-12 (local) of the largest
component in FP64, 1e-4 in FP32."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle.forces import local_force, nonlocal_force
from paper_1603_04339_amd import sparc as sp
from paper_1603_04339_amd import workloads as wl
from tests.helpers import oracle_setup, to_dev

pytestmark = pytest.mark.gpu

TYPES = {"r64": (sp.R64, torch.float64, 1e-11), "r32": (sp.R32, torch.float32, 1e-4),
         "c128": (sp.C128, torch.complex128, 1e-11), "c64": (sp.C64, torch.complex64, 1e-4)}


@pytest.fixture(scope="module")
def ctx():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    c = sp.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("dt", list(TYPES))
@pytest.mark.parametrize("n,n_o", [((13, 14, 15), 6), ((21, 17, 16), 6), ((21, 17, 16), 5)])
@pytest.mark.parametrize("ls", [(0,), (0, 1)])
def test_nonlocal_force(ctx, n, n_o, ls, dt):
    code, tdt, tol = TYPES[dt]
    cplx = dt.startswith("c")
    k = (0.17, -0.11, 0.23) if cplx else (0.0, 0.0, 0.0)
    cell, rng = wl.draw_cell(99, sum(n), n, tuple(0.5 * v for v in n), 5, ls, 2.2, 0)
    grid, V, P = oracle_setup(cell, k, n_o)
    ns = 19
    A = rng.standard_normal((grid.n_d, ns)) + (1j * rng.standard_normal((grid.n_d, ns)) if cplx else 0.0)
    Xd = to_dev(np.ascontiguousarray(np.linalg.qr(A)[0].T), tdt)
    X = Xd.cpu().numpy().T.astype(np.complex128 if cplx else np.float64)
    occ = rng.uniform(0.1, 1.0, ns)
    occ[[2, 9, 10, 18]] = 0.0
    Xd[[2, 9, 10, 18]] = float("nan")
    ham = sp.Hamiltonian(ctx, cell, code, n_o=n_o, kpt=k)
    F = torch.zeros(len(cell.depth), 3, dtype=torch.float64, device="cuda")
    sp.forces_nonlocal(ham, Xd, to_dev(occ), F, sp.workspace(ham, ns, sp.OP_FORCES))
    ref = nonlocal_force([grid], [P], [X], occ[None, :], len(cell.depth))
    assert np.abs(F.cpu().numpy() - ref).max() <= tol * np.abs(ref).max()


@pytest.mark.parametrize("n,h", [((12, 13, 14), 0.4), ((20, 16, 18), 0.7), ((40, 17, 33), 1.6)])
def test_local_force(ctx, n, h):
    cell, rng = wl.draw_cell(99, n[0], n, tuple(h * v for v in n), 3, (0,), 1.5, 0)
    grid, V, P = oracle_setup(cell)
    rho = rng.uniform(0.0, 0.5, grid.n_d)
    ham = sp.Hamiltonian(ctx, cell, sp.R64)
    F = torch.zeros(len(cell.depth), 3, dtype=torch.float64, device="cuda")
    sp.forces_local(ham, to_dev(rho), F)
    ref = local_force(grid, cell.positions, cell.depth, cell.width, rho)
    assert np.abs(F.cpu().numpy() - ref).max() <= 1e-12 * np.abs(ref).max()
